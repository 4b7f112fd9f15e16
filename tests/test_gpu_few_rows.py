"""Few rows. The LM head of up to 32 (a stream over the weights) beside the
tiled one: both sides of the line, one and two row groups, the three chunk
forms of the vocabulary (multiples of 128, of 64, neither), and both weight
storages, which must agree bit for bit. Bar: 2e-2 per token, the bar of the
fp16-operand path. The layers of up to 8 rows."""
import numpy as np
import pytest

import oracle
from paper_2601_01513_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [1152, 1088, 1000])
@pytest.mark.parametrize("lens", [[1, 0], [9, 7], [16, 1], [16, 16], [16, 17]])
def test_lm_head_of_few_rows(vocab, lens):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01513_amd.binding import Verifier
    cfg = W.VerifierConfig(
        name=f"few rows V{vocab} {lens}", n_layers=1, d_model=256, n_heads=2, n_kv_heads=1,
        head_dim=128, d_ff=128, vocab=vocab, rope_base=1e6, dtype=W.BF16, n_prefix=40,
        n_visual=8, n_cands=2, cand_len=17)
    wl = W.make_workload(cfg, sum(lens), device="cuda")
    wl.cand_ids[0, 0] = vocab - 1  # a target in the last chunk
    for m in range(2):
        wl.cand_ids[m, lens[m]:] = 0
    lens = np.asarray(lens, dtype=np.int32)
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda")
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    out = []
    for storage in ("f16", "bf16"):
        v = Verifier(cfg, wl.weights, device="cuda", gemm_weights=storage)
        v.prefill(wl.visual, ids)
        out.append([t.cpu().numpy() for t in v.score(cids, lens)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    ref, sc, am = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                             W.to_host_f32(wl.visual), wl.prefix_ids,
                                             wl.cand_ids, lens)
    assert np.abs(out[0][0] - ref).max() <= 2e-2
    assert int(out[0][2][0]) == am or abs(sc[0] - sc[1]) < 0.1


@pytest.mark.parametrize("d, rows", [(2048, 32), (2048, 33), (2112, 24), (2112, 25), (2560, 25),
                                     (2624, 25), (4096, 24), (4160, 16), (4160, 17), (4160, 128)])
def test_lm_head_lines(d, rows):
    """Both sides of the lines between the stream and the tiles (rows, by width)
    and between the tiles of up to 128 rows (width 2560, fp16 weights): the weight
    storages, which take different tiles, agree bit for bit."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01513_amd.binding import Verifier
    cfg = W.VerifierConfig(
        name=f"head d{d} rows {rows}", n_layers=1, d_model=d, n_heads=1, n_kv_heads=1,
        head_dim=128, d_ff=64, vocab=1088, rope_base=1e6, dtype=W.BF16, n_prefix=20, n_visual=4,
        n_cands=2, cand_len=rows)
    wl = W.make_workload(cfg, rows, device="cuda")
    lens = np.asarray([rows - 1, 1], dtype=np.int32)
    wl.cand_ids[1, 1:] = 0
    wl.cand_ids[0, 0] = cfg.vocab - 1
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda")
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    out = []
    for storage in ("f16", "bf16"):
        v = Verifier(cfg, wl.weights, device="cuda", gemm_weights=storage)
        v.prefill(wl.visual, ids)
        out.append(v.score(cids, lens)[0].cpu().numpy())
    np.testing.assert_array_equal(out[0], out[1])
    ref, _, _ = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                           W.to_host_f32(wl.visual), wl.prefix_ids,
                                           wl.cand_ids, lens)
    assert np.abs(out[0] - ref).max() <= 2e-2


# (d_model, heads, d_ff): the loads a wave's lanes make per weight row and the
# waves left without any: 4 pairs of K for 16 waves; a long down projection on
# few outputs; more than 256 output groups in several steps.
@pytest.mark.parametrize("d, hq, ff", [(256, 2, 320), (256, 2, 6464), (2112, 3, 7104)])
@pytest.mark.parametrize("prefix, lens", [(40, [1, 0]), (40, [7, 1]), (40, [8, 1]), (4, [3, 0])])
def test_layers_of_few_rows(d, hq, ff, prefix, lens):
    """Layers of up to 8 rows in one launch per projection (8 and 9 rows: both
    sides of the line; 4 prefix rows: the fused pass itself is one), with split
    operands in no, the attention's and both halves of the first layer. Fused
    and two-call passes and both storages run the same products."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01513_amd.binding import Verifier
    cfg = W.VerifierConfig(
        name=f"few rows d{d} F{ff}", n_layers=2, d_model=d, n_heads=hq, n_kv_heads=1,
        head_dim=128, d_ff=ff, vocab=512, rope_base=1e6, dtype=W.BF16, n_prefix=prefix,
        n_visual=2, n_cands=2, cand_len=8)
    wl = W.make_workload(cfg, sum(lens), device="cuda")
    for m in range(2):
        wl.cand_ids[m, lens[m]:] = 0
    lens = np.asarray(lens, dtype=np.int32)
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda")
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    ref, sc, am = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                             W.to_host_f32(wl.visual), wl.prefix_ids,
                                             wl.cand_ids, lens)
    for split in ((0, 0), (1, 0), (2, 1)):
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


def test_gains_at_any_address():
    """Norm gains that start 2 bytes into an allocation: the rows that read them
    16 bytes at a time otherwise take the form that does not."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01513_amd.binding import Verifier
    cfg = W.VerifierConfig(
        name="gains off 16 bytes", n_layers=2, d_model=256, n_heads=2, n_kv_heads=1,
        head_dim=128, d_ff=320, vocab=512, rope_base=1e6, dtype=W.BF16, n_prefix=20,
        n_visual=2, n_cands=1, cand_len=6)
    wl = W.make_workload(cfg, 3, device="cuda")
    ids = torch.tensor(wl.prefix_ids, dtype=torch.int32, device="cuda")
    cids = torch.tensor(wl.cand_ids, dtype=torch.int32, device="cuda")
    ref, _, _ = oracle.score_shared_prefix(cfg, W.host_weights(wl.weights),
                                           W.to_host_f32(wl.visual), wl.prefix_ids, wl.cand_ids,
                                           wl.cand_len)
    for lw in wl.weights["layers"]:
        for k in ("attn_norm", "ffn_norm"):
            off = torch.empty(cfg.d_model + 1, dtype=lw[k].dtype, device="cuda")[1:]
            lw[k] = off.copy_(lw[k])
            assert lw[k].data_ptr() % 16 == 2
    v = Verifier(cfg, wl.weights, device="cuda")
    v.prefill(wl.visual, ids)
    assert np.abs(v.score(cids, wl.cand_len)[0].cpu().numpy() - ref).max() <= 2e-2
