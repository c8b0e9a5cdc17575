"""GPU parity of the paper's coarse query-frame evidence
(evisel_coarse_evidence: appendix, coarse-map equation) and a synthetic
analogue of the sparse-vs-dense alignment table (Reliability of Sparse
Attention Maps) computed from the GPU's maps.

Coarse evidence is compared with the oracle on every frame: tolerance 1e-4
(fp32: 1e-5), and on top what the rows can add whose cut lies within the
kernel's rounding in the oracle (see the top-p tests for that margin): the
mass of the blocks that such a row may keep or drop, on those blocks' frames,
and its share of the row's other mass. That sum has to stay a small part of
the evidence.

The alignment test computes Pearson, Spearman, JS, Top-10 %, Keep and
Mass-recovery of the exact sparse cues (A_qf, A_ff, A_if) and of the coarse
A_qf against dense causal attention, once from the GPU's maps and once from
the oracle's sparse maps, and requires the two to agree; it prints the
table.
"""
import numpy as np
import pytest

from oracle import coarse, cues, topp
from oracle.layout import Layout, VIS
import workloads as wl
from gpu_harness import run_gpu, to_device, say
from test_gpu_topp import _gpu_bits, _keep_of_rows, TAU

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    pytest.ev = gpu_lib


def _w(name, **kw):
    base = dict(name=name, config_id=901, n_layers=1, hq=4, hkv=2, d=128,
                dtype="bf16", tokens_per_frame=32, block=64, sink_blocks=1,
                window=8, plant="choose", tau_p=TAU,
                plant_args={"count": 3, "s_frame": (2.0, 3.0),
                            "s_query": 2.0})
    base.update(kw)
    return wl.Workload(**base)


CASES = {
    "ragged_struct": _w("ragged-struct", n_frames=(9, 14, 5),
                        n_text=(64, 32, 130), n_sys=(5, 0, 70), n_videos=3,
                        key_struct=(2.0, 2.0, 0.8)),
    "fp32_d64": _w("fp32-d64", dtype="fp32", d=64, hq=4, hkv=1,
                   tokens_per_frame=16, n_frames=(40,), n_text=(48,),
                   n_sys=(3,), key_struct=(2.0, 2.0, 0.8)),
    "plain_d64": _w("plain-d64", d=64, hq=8, hkv=2, tokens_per_frame=64,
                    n_frames=(24,), n_text=(100,), n_sys=(0,)),
    "config2": wl.get(2, tau_p=TAU),
}


# The query rows' histories at the edges of a wave's share (one row per wave, a
# block per lane, four steps of 64 blocks at a time): one block, one group of
# steps and the next, a short last visual block, and the longest history a mask
# accepts (2,047 blocks, with one to spare for the row's own).
EDGES = {
    "one_block": _w("one-block", n_frames=(1,), n_text=(3,), n_sys=(0,),
                    plant_args={"count": 1, "s_frame": (2.0, 3.0),
                                "s_query": 2.0}),
    "share_4": _w("share-4", hq=2, tokens_per_frame=64, n_frames=(256,),
                  n_text=(17,), n_sys=(0,)),
    "share_8_short": _w("share-8-short", hq=2, tokens_per_frame=16,
                        n_frames=(1027,), n_text=(80,), n_sys=(65,)),
    "fp32_share_8": _w("fp32-share-8", dtype="fp32", hq=2, hkv=1,
                       tokens_per_frame=64, n_frames=(300,), n_text=(5,),
                       n_sys=(130,)),
    "longest": _w("longest", d=64, hq=2, tokens_per_frame=64,
                  n_frames=(2046,), n_text=(70,), n_sys=(0,)),
}


# System prefixes: their blocks and the history's share a work-group's 16 waves
# by number (at least one each), both with one tile and with many.
PREFIX = {
    "one_each": _w("one-each", n_frames=(4,), n_text=(17,), n_sys=(64,)),
    "waves_15": _w("waves-15", hq=2, hkv=1, n_frames=(4,), n_text=(65,),
                   n_sys=(961,)),
    "long": _w("long-prefix", hq=2, hkv=1, tokens_per_frame=16, n_frames=(5,),
               n_text=(70,), n_sys=(4159,)),
    "shared_d64": _w("shared-d64", d=64, hq=2, hkv=1, tokens_per_frame=64,
                     n_frames=(300,), n_text=(20,), n_sys=(1100,)),
    "fp32_long": _w("fp32-long", dtype="fp32", hq=2, hkv=1, n_frames=(3,),
                    n_text=(33,), n_sys=(2050,)),
    "fp32_d64": _w("fp32-prefix-d64", dtype="fp32", d=64, hq=2, hkv=1,
                   n_frames=(70,), n_text=(64,), n_sys=(300,)),
}


def _layout(w):
    ns, nf, nt = wl.layout_arrays(w)
    return Layout(ns, nf, nt, w.tokens_per_frame)


def _gpu_coarse(w, mask, l=0, inputs=None):
    import torch
    ev = pytest.ev
    q, k, _ = to_device(inputs or wl.gen_layer(w, l), w, torch)
    T = mask.stats["n_frames_total"]
    out = torch.full((w.hq, T), float("nan"), device="cuda")
    ws = torch.empty(ev.sparse_prefill_workspace(mask, w.d),
                     dtype=torch.uint8, device="cuda")
    ev.coarse_evidence(mask, q, k, out, ws, softmax_scale=w.softmax_scale)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("name", list(EDGES))
def test_coarse_evidence_history_edges(name):
    _check_coarse(name, EDGES[name])


@pytest.mark.parametrize("name", list(PREFIX))
def test_coarse_evidence_system_prefix(name):
    _check_coarse(name, PREFIX[name])


@pytest.mark.parametrize("name", ["share_4", "share_8_short", "fp32_share_8"])
def test_coarse_evidence_ties(name):
    """All affinities equal (Q = 0): the lowest blocks are kept."""
    w = EDGES[name]
    _check_coarse(name, w, wl.gen_layer(w, 0, q_override="zero"), ties=True)


# Equal affinities at the cut beside blocks so far below that exp2 of their
# difference is +0: the zeros are no ties and take no part in the count.
# (tau, blocks at 0, blocks at about -6.9, blocks at -200 nats); the dropped
# mass (1 - tau) Z is no multiple of a tie's, so the cut is not at rounding.
UNDERFLOW = [(0.97, 64, 0, 10), (0.97, 64, 0, 1), (0.97, 64, 0, 2),
             (0.97, 90, 0, 300), (0.5, 101, 0, 100), (0.97, 1, 100, 40),
             (0.97, 1, 100, 1), (0.9, 3, 2000, 40), (0.97, 1, 0, 70)]


@pytest.mark.parametrize("case", UNDERFLOW)
def test_coarse_evidence_ties_beside_underflow(case):
    tau, n_top, n_mid, n_far = case
    ev = pytest.ev
    F = n_top + n_mid + n_far
    w = _w("underflow", d=64, hq=2, hkv=1, tokens_per_frame=64, n_frames=(F,),
           n_text=(21,), n_sys=(0,), tau_p=float(np.float32(tau)),
           plant_args={"count": 1, "s_frame": (2.0, 3.0), "s_query": 2.0})
    inputs = wl.gen_layer(w, 0)
    # affinity 16 k[0] / sqrt(64), in values that bf16 holds exactly
    level = np.repeat([0.0, -3.453125, -100.0], [n_top, n_mid, n_far])
    level = np.random.default_rng(3).permutation(level)
    bf = lambda a: (a.astype(np.float32).view(np.uint32) >> 16).astype(
        inputs.q.dtype)
    q, k = np.zeros(inputs.q.shape), np.zeros(inputs.k.shape)
    q[..., 0] = 16.0
    k[:64 * F, 0, 0] = np.repeat(level, 64)
    inputs.q, inputs.k = bf(q), bf(k)
    lay = _layout(w)
    blk = topp.Blocks(lay, w.block)
    mask = ev.build_block_mask([F], [21], 64, 64, 1, 8, 2, 1, tau_p=w.tau_p)
    Eg = _gpu_coarse(w, mask, inputs=inputs)
    q, k, _ = inputs.as_f64()
    txt = lay.text_rows()
    keep, _ = topp.select(q, k, lay, blk, w.tau_p, w.softmax_scale, txt)
    rb, _ = _gpu_bits(ev, mask, w, 0, inputs=inputs)
    kg = _keep_of_rows(ev, rb, mask, blk, txt, keep.shape[2])
    Eo = coarse.query_frame(lay, coarse.coarse_probs(
        q, k, lay, blk, keep, txt, w.softmax_scale), w.hq)
    say(f"  kept {int(keep[0, 0].sum())} of {F}, by the selection "
        f"{int(kg[0, 0].sum())}, by the coarse pass {int((Eg[0] > 0).sum())}")
    # every row is the same: a frame has mass where its block is kept
    assert (keep == keep[:1, :1]).all()
    seen = level > -100.0                      # the others' mass is below 1e-80
    assert ((Eg > 0) == (keep[:, 0, :F] & seen)).all()
    assert (kg[:, :, :F][:, :, seen] == keep[:, :, :F][:, :, seen]).all()
    assert np.abs(Eg - Eo).max() <= 1e-5 * Eo.max()


def test_coarse_evidence_all_affinities_minus_infinite():
    """Query rows whose every block affinity overflows to -inf put no mass on
    the history."""
    w = _w("minus-inf", d=64, hq=2, hkv=1, tokens_per_frame=32, n_frames=(9,),
           n_text=(21,), n_sys=(0,))
    inputs = wl.gen_layer(w, 0)
    bf = lambda x: np.float32(x).view(np.uint32) >> 16
    n = 9 * 32
    inputs.k[:, :, 0] = 0
    inputs.k[:n, :, 0] = bf(-1e10)
    inputs.q[n:, :, 0] = bf(1e30)
    mask = pytest.ev.build_block_mask([9], [21], 32, 64, 1, 8, 2, 1,
                                      tau_p=w.tau_p)
    assert (_gpu_coarse(w, mask, inputs=inputs) == 0).all()


@pytest.mark.parametrize("name", list(CASES))
def test_coarse_evidence(name):
    _check_coarse(name, CASES[name])


def _flip_bound(q, k, lay, blk, txt, keep, info, groups, w):
    """[Hq, T]: how far rows whose cut lies within the kernel's rounding can
    move each frame's evidence, from the oracle alone."""
    kbar = topp.mean_keys(k, blk)
    grp = w.hq // w.hkv
    B = np.zeros((w.hq, lay.T))
    at = {int(i): j for j, i in enumerate(txt)}
    u_aff = 2.0 ** -16 + (2 * w.d + 70) * 2.0 ** -24
    for ri, keys, P in groups:
        n, lb = int(lay.seq[ri[0]]), int(blk.local[ri[0]])
        if lb <= 0:
            continue
        hist = kbar[blk.first[n]:blk.first[n] + lb]
        local, frame = blk.local[keys], lay.frame[keys]
        on_hist = (local >= 0) & (local < lb)
        lens = np.bincount(local[on_hist], minlength=lb)[:lb]
        for h in range(w.hq):
            g = q[ri, h] @ hist[:, h // grp].T * w.softmax_scale
            p = np.exp(g - g.max(1, keepdims=True))
            p /= p.sum(1, keepdims=True)
            bound = (np.abs(q[ri, h]) @ np.abs(hist[:, h // grp]).T).max(
                1) * w.softmax_scale
            for r, i in enumerate(ri):
                j = at[int(i)]
                e = 2 * bound[r] * u_aff + 1e-6
                ec = 2 * e + lb * 2.0 ** -23
                pl, pn = info["p_last"][h, j], info["p_next"][h, j]
                before = info["c_before"][h, j] > w.tau_p - ec
                after = info["c_at"][h, j] < w.tau_p + ec
                near = pn >= 0 and pl - pn < 2 * e * pl
                if not (before or after or near):
                    continue
                low = pn if pn >= 0 and (after or near) else pl
                flip = (p[r] >= low * (1 - 2 * e)) & (p[r] <= pl * (1 + 2 * e))
                # a block's mass per unit of len * p, from the row's own
                kept = keep[h, j, :lb]
                per = P[h, r][on_hist].sum() / (lens * p[r] * kept).sum()
                mass = np.where(flip, lens * p[r] * per, 0.0)
                blk_mass = np.where(on_hist, mass[np.maximum(local, 0) % lb]
                                    / lens[np.maximum(local, 0) % lb], 0.0)
                vis = frame >= 0
                B[h] += np.bincount(frame[vis], weights=(
                    blk_mass + P[h, r] * mass.sum())[vis], minlength=lay.T)
    return B


def _check_coarse(name, w, inputs=None, ties=False):
    """``ties``: every affinity is exactly equal, so no row is at rounding but
    those whose tau_p * blocks is a whole number, nearly."""
    ev = pytest.ev
    say(f"case {name}")
    lay = _layout(w)
    blk = topp.Blocks(lay, w.block)
    ns, nf, nt = wl.layout_arrays(w)
    mask = ev.build_block_mask(nf, nt, w.tokens_per_frame, w.block,
                               w.sink_blocks, w.window, w.hq, w.hkv,
                               n_sys=ns, tau_p=w.tau_p)
    inputs = inputs or wl.gen_layer(w, 0)
    Eg = _gpu_coarse(w, mask, inputs=inputs)
    q, k, _ = inputs.as_f64()
    txt = lay.text_rows()
    keep, info = topp.select(q, k, lay, blk, w.tau_p, w.softmax_scale, txt)
    groups = coarse.coarse_probs(q, k, lay, blk, keep, txt, w.softmax_scale)
    Eo = coarse.query_frame(lay, groups, w.hq)
    B = np.zeros_like(Eo) if ties else _flip_bound(q, k, lay, blk, txt, keep,
                                                   info, groups, w)
    err = np.abs(Eg - Eo)
    say(f"  coarse evidence err {err.max():.2e}, rows at rounding "
        f"{B.max():.2e} at most, {B.sum() / Eo.sum():.2e} of the mass")
    assert np.isfinite(Eg).all()
    assert B.sum() <= 0.05 * Eo.sum()
    assert (err <= (1e-5 if w.dtype == "fp32" else 1e-4) + B).all()


def test_alignment_table():
    w = _w("align", n_frames=(48,), n_text=(64,), n_sys=(0,), hq=4, hkv=2,
           key_struct=(2.0, 2.0, 0.8))
    ev = pytest.ev
    lay = _layout(w)
    blk = topp.Blocks(lay, w.block)
    res = run_gpu(ev, w, [0], cues=True, keep_o=False)
    E_coarse = _gpu_coarse(w, res.mask)
    q, k, v = wl.gen_layer(w, 0).as_f64()
    rows = np.arange(lay.S)
    vis = np.nonzero(lay.region == VIS)[0]
    keep, _ = topp.select(q, k, lay, blk, w.tau_p, w.softmax_scale, rows)
    # oracle sparse (exact), coarse and dense maps
    sp = list(cues.topp_groups(q, k, v, lay, blk, keep, rows,
                               w.softmax_scale))
    co = coarse.coarse_probs(q, k, lay, blk, keep, rows, w.softmax_scale)
    de = list(coarse.dense_groups(q, k, v, lay, rows, w.softmax_scale))

    def maps(groups):
        g = list(groups)
        E = coarse.query_frame(lay, g, w.hq).sum(axis=0)
        A_ff, A_if = cues.accumulate(
            lay, [(r[lay.region[r] == VIS], kk, P[:, lay.region[r] == VIS])
                  for r, kk, P in g], w.hq)
        return E, A_ff, A_if
    Es, FFs, IFs = maps(sp)
    Ec, _, _ = maps(co)
    Ed, FFd, IFd = maps(de)
    tri = np.tril(np.ones((lay.T, lay.T), bool), -1)
    low = np.tril(np.ones((w.tokens_per_frame,) * 2, bool))[None]
    low = np.broadcast_to(low, IFd.shape)
    # the GPU's maps
    A_ff_g = np.zeros((lay.T, lay.T))
    pr = ev.mask_export_pairs(res.mask)
    A_ff_g[pr["a"], pr["b"]] = res.pairs[0]
    gpu = {"A_qf": res.E[0].sum(axis=0), "A_ff": A_ff_g[tri],
           "A_if": res.intra[0][low], "A_qf coarse": E_coarse.sum(axis=0)}
    ora = {"A_qf": Es, "A_ff": FFs[tri], "A_if": IFs[low], "A_qf coarse": Ec}
    dense = {"A_qf": Ed, "A_ff": FFd[tri], "A_if": IFd[low],
             "A_qf coarse": Ed}
    say("  cue          Pear.   Spear.  JS       Top-10%  Keep    Mass-rec")
    for name in gpu:
        mg = coarse.alignment(gpu[name], dense[name])
        mo = coarse.alignment(ora[name], dense[name])
        say(f"  {name:12s} {mg['pearson']:.3f}   {mg['spearman']:.3f}   "
            f"{mg['js']:.4f}   {mg['top10']:.3f}    {mg['keep']:.3f}   "
            f"{mg['mass_rec']:.4f}")
        for key in ("pearson", "spearman", "mass_rec"):
            assert abs(mg[key] - mo[key]) <= 5e-3, (name, key)
        assert abs(mg["js"] - mo["js"]) <= 1e-3
        assert abs(mg["keep"] - mo["keep"]) <= 2.0 / gpu[name].size
        assert abs(mg["top10"] - mo["top10"]) <= 0.1
