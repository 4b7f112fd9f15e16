"""Edges of the dispatches of the retrieval stage and of the entity alignment,
against float64 or integer references computed here: parts of a frame, frames
that start at every byte alignment, more than 64 frames per keyframe thread,
groups of 16 and of 32 keyframes, side by side and in turn, widths with a
partial last piece and unaligned rows, several batches of documents per block,
and both forms of the alignment on either side of their line.

Bars: counts and indices exact; similarities within 1e-6 (float32 sums of at
most 900 terms of a unit vector product: n eps / 2 is 5e-5 in the worst case,
sqrt(n) eps about 2e-6 times a cosine below 0.5)."""
import numpy as np
import pytest

from oracle import retrieval as R

pytestmark = pytest.mark.gpu
TOL = 1e-6


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("nf,h,w", [(3, 150, 161), (5, 256, 256), (2, 1, 30000), (127, 149, 148),
                                    (130, 149, 149), (16, 7, 3), (1500, 2, 3), (65, 1, 1),
                                    (130, 224, 224), (170, 401, 401), (171, 401, 401)])
def test_keyframes_against_counts(nf, h, w):
    torch = _torch()
    from paper_2601_01513_amd.binding import Retriever
    rng = np.random.default_rng(nf)
    frames = rng.integers(0, 256, size=(nf, h, w, 3)).astype(np.uint8)
    frames[nf // 2:] //= 8  # a cut
    r = Retriever(nf, h, w, 1, 1, 1, 1)
    key_idx, n_keys = r.keyframes(torch.tensor(frames, device="cuda"), 0.6)
    hist = np.zeros((nf, 3, 64), dtype=np.int64)
    for f in range(nf):
        for c in range(3):
            hist[f, c] = np.bincount(frames[f, :, :, c].ravel() >> 2, minlength=64)
    inter = np.minimum(hist[1:], hist[:-1]).sum(axis=(1, 2))
    thr = float(np.float32(0.6)) * 3.0 * (h * w)
    keys = np.concatenate([[0], 1 + np.nonzero(inter < thr)[0]])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(r.hist.cpu().numpy(), hist)
    np.testing.assert_array_equal(r.inter.cpu().numpy()[1:], inter)
    assert int(r.inter.cpu()[0]) == -1
    assert int(n_keys.cpu()[0]) == len(keys)
    np.testing.assert_array_equal(key_idx.cpu().numpy()[:len(keys)], keys)


def _scan_plan(nf, nk, nd, dim):
    """The bank scan's launch: keyframes per pass, passes of the busiest block,
    batches (at most 256 documents each) of the largest share."""
    row = ((dim + 15) // 16 * 16 + 4) * 4
    wide = nf > 16 and 32 * (row + 1024) <= 150 << 10
    rows = 32 if wide else 16
    nlists = min((nd + 255) // 256, 256)
    ny = min((nf + 15) // 16, 256 // nlists)
    if nk <= 16 * ny:
        rows = 16
    groups = (nk + rows - 1) // rows
    return rows, (groups + ny - 1) // ny, (-(-nd // nlists) + 255) // 256


# `plan`: keyframes per pass, passes, batches.
@pytest.mark.parametrize("nf,nk,nd,dim,k,K,plan", [
    (12, 12, 513, 48, 2, 3, (16, 1, 1)),       # one group of 16, aligned
    (40, 16, 300, 35, 3, 5, (16, 1, 1)),       # unaligned rows, a partial piece
    (40, 17, 300, 36, 16, 64, (16, 1, 1)),     # two groups side by side
    (70, 70, 2000, 100, 5, 40, (16, 1, 1)),    # five
    (40, 40, 700, 900, 3, 9, (16, 1, 1)),      # long rows
    (40, 40, 66000, 900, 3, 9, (32, 2, 2)),    # ... and more documents than one batch each
    (20, 20, 65001, 20, 4, 8, (32, 1, 1)),     # the second 16 of a group of 32
    (70, 70, 65001, 20, 4, 8, (32, 3, 1)),     # three groups of 32 in turn
    (300, 200, 90, 13, 16, 64, (16, 1, 1)),    # more than 1024 entries to select from
    (300, 300, 20000, 13, 2, 9, (32, 4, 1)),   # groups of 32 side by side and in turn
    (40, 40, 22000, 944, 3, 9, (16, 2, 1)),    # rows too long for 32: groups of 16 in turn
    (3, 1, 1, 1, 1, 1, (16, 1, 1)),
    # Several batches, the wave's second tile in use in every other one (128 and
    # 129 documents), its stored list merged, in a second group as well.
    (40, 40, 256 * 257, 20, 4, 8, (32, 2, 2)),
    (16, 16, 256 * 257, 20, 4, 8, (16, 1, 2)),
])
def test_retrieve_groups(nf, nk, nd, dim, k, K, plan):
    assert _scan_plan(nf, nk, nd, dim) == plan
    torch = _torch()
    from paper_2601_01513_amd.binding import Retriever
    g = torch.Generator(device="cuda")
    g.manual_seed(nf * 7 + nd)
    femb = torch.randn((nf, dim), generator=g, device="cuda")
    docs = torch.randn((nd, dim), generator=g, device="cuda")
    r = Retriever(nf, 1, 1, nd, dim, k, K)
    keys = torch.arange(nf - 1, nf - 1 - nk, -1, device="cuda").int()
    r.key_idx[:nk] = keys
    r.n_keys.fill_(nk)
    top_idx, top_sim, sel_idx, sel_sim, n_sel = r.retrieve(femb, docs)
    torch.cuda.synchronize()
    kk = min(k, nd)
    idx, sim = top_idx[:nk].cpu().numpy(), top_sim[:nk].cpu().numpy()
    sims = R.cosine_matrix(femb[keys.long()].cpu().numpy(), docs.cpu().numpy())
    best = {}
    for i in range(nk):
        order = R.top_indices(sims[i], k)
        np.testing.assert_allclose(sim[i, :kk], sims[i][order], rtol=0, atol=TOL)
        np.testing.assert_allclose(sims[i][idx[i, :kk]], sims[i][order], rtol=0, atol=TOL)
        assert len(set(idx[i, :kk].tolist())) == kk and np.all(idx[i, kk:] == -1)
        for d, v in zip(idx[i, :kk].tolist(), sim[i, :kk].tolist()):
            best[d] = max(best.get(d, -2.0), v)
    # T* from the lists themselves: exact, ties to the lower index.
    want = sorted(best.items(), key=lambda e: (-e[1], e[0]))[:K]
    n = int(n_sel.cpu()[0])
    assert n == len(want)
    assert sel_idx.cpu().numpy()[:n].tolist() == [d for d, _ in want]
    np.testing.assert_array_equal(sel_sim.cpu().numpy()[:n],
                                  np.array([v for _, v in want], dtype=np.float32))


@pytest.mark.parametrize("dim", [100, 500, 768, 1000])
def test_similarities_keep_their_bits(dim):
    """2-norm error of the similarities found over 20 banks: sums of at most dim / 4
    terms in four chains, measured 0.8e-7 to 1.4e-7 for 33 to 1024 dimensions (one
    chain over all of them: 1.6e-7 to 4.7e-7)."""
    torch = _torch()
    from paper_2601_01513_amd.binding import Retriever
    g = torch.Generator(device="cuda")
    g.manual_seed(dim)
    err = ref = 0.0
    for _ in range(20):
        femb = torch.randn((8, dim), generator=g, device="cuda")
        docs = torch.randn((300, dim), generator=g, device="cuda")
        docs[:8] += femb  # each keyframe has a near document, as in a real bank
        r = Retriever(8, 1, 1, 300, dim, 8, 8)
        r.key_idx.copy_(torch.arange(8, device="cuda"))
        r.n_keys.fill_(8)
        idx, sim, _, _, _ = r.retrieve(femb, docs)
        q, d = femb.double(), docs.double()
        s = (q / q.norm(dim=1, keepdim=True)) @ (d / d.norm(dim=1, keepdim=True)).T
        want = s.gather(1, idx.long())
        err += (sim.double() - want).square().sum().item()
        ref += want.square().sum().item()
    assert (err / ref) ** 0.5 <= (1.4e-7 if dim == 100 else 2e-7)


def test_small_bank_takes_many_keyframes_side_by_side():
    """200 keyframes against a question's own 156 documents: about 1.1 times the
    time of 16 (38 and 35 us); their groups one after the other took 8 times."""
    torch = _torch()
    from paper_2601_01513_amd.binding import Retriever
    femb, docs = torch.randn((200, 768), device="cuda"), torch.randn((156, 768), device="cuda")

    def us(nk):
        r = Retriever(200, 1, 1, 156, 768, 3, 5)
        r.key_idx.copy_(torch.arange(200, device="cuda"))
        r.n_keys.fill_(nk)
        runs = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                r.retrieve(femb, docs)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b) * 50.0)
        return min(runs)

    assert us(200) < 2.5 * us(16)


@pytest.mark.parametrize("strategy", ["two_stage", "addition", "invert"])
@pytest.mark.parametrize("M,NF,D", [(7, 192, 33), (7, 193, 33), (17, 200, 16), (16, 65, 770),
                                    (256, 193, 4), (1, 5000, 3), (33, 1025, 129)])
def test_align_both_forms(M, NF, D, strategy):
    torch = _torch()
    from paper_2601_01513_amd.binding import align_select
    g = torch.Generator(device="cuda")
    g.manual_seed(M + NF)
    # Rows start at odd 4-byte addresses.
    ent = torch.randn(M * D + 1, generator=g, device="cuda")[1:].view(M, D)
    frames = torch.randn(NF * D + 3, generator=g, device="cuda")[3:].view(NF, D)
    ent[M // 2] = 0.0
    rel = torch.rand(M, generator=g, device="cuda")
    align, choice = align_select(ent, frames, rel, 0.05, strategy)
    e, f = ent.double().cpu().numpy(), frames.double().cpu().numpy()
    en, fn = np.linalg.norm(e, axis=1), np.linalg.norm(f, axis=1)
    den = en[:, None] * fn[None, :]
    ref = np.where(den > 0, (e @ f.T) / np.where(den > 0, den, 1.0), 0.0).max(axis=1)
    a, r = align.cpu().numpy(), rel.cpu().numpy()
    np.testing.assert_allclose(a, ref, rtol=0, atol=TOL)
    # The choice is the rule's on the returned float32 values.
    if strategy == "addition":
        want = int(np.argmax(r + a))
    else:
        filt, rank = (r, a) if strategy == "two_stage" else (a, r)
        ok = filt >= filt.max() - np.float32(0.05)
        want = int(np.argmax(np.where(ok, rank, -np.inf)))
    assert int(choice.cpu()[0]) == want


@pytest.mark.parametrize("M,NF,D", [(8, 64, 768), (8, 300, 768), (64, 2048, 1024)])
def test_alignments_keep_their_bits(M, NF, D):
    """2-norm error of the alignments over 20 draws: 7.4e-8 to 7.7e-8 in both forms
    (the tiled one as one chain per wave: 1.4e-7 to 1.6e-7)."""
    torch = _torch()
    from paper_2601_01513_amd.binding import align_select
    g = torch.Generator(device="cuda")
    g.manual_seed(NF)
    err = ref = 0.0
    for _ in range(20):
        ent = torch.randn((M, D), generator=g, device="cuda")
        frames = torch.randn((NF, D), generator=g, device="cuda")
        align, _ = align_select(ent, frames, torch.rand(M, device="cuda"), 0.05, "addition")
        e, f = ent.double(), frames.double()
        want = ((e / e.norm(dim=1, keepdim=True)) @ (f / f.norm(dim=1, keepdim=True)).T).amax(1)
        err += (align.double() - want).square().sum().item()
        ref += want.square().sum().item()
    assert (err / ref) ** 0.5 <= 1.1e-7


def test_align_nan_values_keep_their_rule():
    """A NaN rank at the first allowed draft wins (nothing is greater), one
    further on is never chosen; NaN cosines do not enter a maximum."""
    torch = _torch()
    from paper_2601_01513_amd.binding import align_select
    frames = torch.eye(4, device="cuda")
    ent = torch.eye(4, device="cuda")
    nan = float("nan")
    for rel, want in (([nan, 0.5, 0.7, 0.2], 0), ([0.5, nan, 0.7, 0.2], 2)):
        _, choice = align_select(ent, frames, torch.tensor(rel, device="cuda"), 0.05, "addition")
        assert int(choice.cpu()[0]) == want
    ent[1] = nan
    align, choice = align_select(ent, frames, torch.full((4,), 0.5, device="cuda"), 0.05,
                                 "two_stage")
    assert align.cpu().tolist()[0::2] == [1.0, 1.0] and int(choice.cpu()[0]) == 0
