"""Aggregation over layers and heads (evisel_frame_evidence) at the sizes
where its kernels' tiles end, against the oracle's formulas: frame counts
around the 64-frame groups and the 4,096-score chunks of the top-k, ties, NaN
and -inf scores, layer counts around the four-layer groups of E_ff, head counts
with and without each group of the head loop (16, 8, 4, 2, 1)."""
import numpy as np
import pytest

from oracle.cues import e_ff
from oracle.layout import Layout

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    pytest.ev = gpu_lib


CASES = {   # frames per video, k per video, layers, heads
    "one_frame": ((1,), (1,), 1, 1),
    "groups": ((63, 64, 65, 1, 130), (5, 64, 0, 9, 130), 8, 4),
    "chunks": ((4095, 4097, 4161), (300, -3, 5000), 1, 1),
    "layers_15": ((40,), (7,), 15, 28),
    "layers_3_heads_31": ((70, 9), (7, 3), 3, 31),
    "layers_4_heads_12": ((33,), (4,), 4, 12),
    "layers_5_heads_34": ((65,), (65,), 5, 34),
    "layers_33_heads_17": ((20, 66), (2, 8), 33, 17),
    # no video past 64 frames: means and ranks in one work-group per video
    "short_videos": ((64, 33, 1, 32, 31), (5, 40, 1, 0, 31), 35, 4),
}


@pytest.mark.parametrize("name", list(CASES))
def test_aggregation_edges(name):
    import torch
    ev = pytest.ev
    frames, ks, L, hq = CASES[name]
    T, nv = sum(frames), 64
    text = [3 + i for i in range(len(frames))]
    mask = ev.build_block_mask(frames, text, nv, 64, 1, 2, hq, 1)
    rng = np.random.default_rng(7)
    E = rng.random((L, hq, T)).astype(np.float32)
    E[:, :, 1::5] = E[:, :, :1]                       # ties
    if T > 20:
        E[0, 0, 3], E[0, 0, 11], E[0, 0, 17] = np.nan, -np.inf, np.nan
    n_pairs = mask.stats["n_frame_pairs"]
    pr = rng.random((L, max(n_pairs, 1))).astype(np.float32)
    cu = lambda a: torch.from_numpy(a).cuda()
    e_qf, e_l = torch.empty(T, device="cuda"), torch.empty(L, T, device="cuda")
    kept = [min(max(k, 0), f) for k, f in zip(ks, frames)]
    top = torch.full((sum(kept) + 1,), -7, dtype=torch.int32, device="cuda")
    eff = torch.full((L, T), float("nan"), device="cuda")
    ev.frame_evidence(mask, cu(E), L, e_qf, e_qf_layer=e_l,
                      k_per_seq=torch.tensor(ks, dtype=torch.int32).cuda(),
                      topk=top, frame_pairs=cu(pr), e_ff=eff)
    torch.cuda.synchronize()
    nt = np.repeat(text, frames)
    ref = E.astype(np.float64).sum(1) / (hq * nt)
    got = e_l.cpu().numpy()
    # fp32 sums of hq (then L) positive terms
    np.testing.assert_allclose(got, ref, rtol=2e-7 * (hq + 2))
    np.testing.assert_allclose(e_qf.cpu().numpy(), ref.mean(0),
                               rtol=2e-7 * (hq + L + 3))
    # the ranking of the GPU's own scores: value descending, index ascending
    score, flat, off, fo = e_qf.cpu().numpy(), top.cpu().numpy(), 0, 0
    for k, f in zip(kept, frames):
        s = score[fo:fo + f].copy()
        s[np.isnan(s)] = -np.inf
        order = np.argsort(-s, kind="stable")[:k]
        assert (flat[off:off + k] == order).all(), (name, f, k)
        off, fo = off + k, fo + f
    assert flat[off] == -7
    lay = Layout([0] * len(frames), list(frames), text, nv)
    pe, A = ev.mask_export_pairs(mask), np.zeros((T, T))
    for l in range(L):
        A[pe["a"], pe["b"]] = pr[l, :n_pairs]
        np.testing.assert_allclose(eff[l].cpu().numpy(), e_ff(lay, A),
                                   rtol=1e-5, atol=1e-9)
