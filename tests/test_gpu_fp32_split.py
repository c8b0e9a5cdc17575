"""The fp32 attention (three-way bf16 split) where its 32-key half tiles and
its fallback matter, against fp64: block lengths around the halves, both head
dims, and keys whose split is not finite (an infinite key component that gives
the key the logit -inf must leave the rows as if the key were not there), with
few and with more than 64 key tiles per item, under top-p retention and with
the frame cues."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    pytest.ev = gpu_lib


def _reference(q, k, v, vis0, txt0, skip=None, drop=None):
    """Plain causal attention in fp64 (one video, window -1), without the key
    ``skip`` and the (row, key) pairs ``drop``: O, LSE, query rows' mass per
    visual token, probabilities."""
    S, hq, d = q.shape
    grp = hq // k.shape[1]
    s = np.stack([q[:, h] @ k[:, h // grp].T for h in range(hq)]) * d ** -0.5
    s[:, np.triu(np.ones((S, S), bool), 1)] = -np.inf
    if skip is not None:
        s[:, :, skip] = -np.inf
    if drop is not None:
        s[:, drop] = -np.inf
    m = s.max(-1, keepdims=True)
    p = np.exp(s - m)
    z = p.sum(-1, keepdims=True)
    p /= z
    E = p[:, txt0:, vis0:txt0].sum(1)
    O = np.stack([p[h] @ v[:, h // grp] for h in range(hq)], 1)
    return O, (m + np.log(z))[..., 0], E, p


def _run(q, k, v, F, nv, nt, ns, tau=0.0, cues=False):
    import torch
    ev = pytest.ev
    S, hq, d = q.shape
    mask = ev.build_block_mask([F], [nt], nv, 64, 1, -1, hq, k.shape[1],
                               n_sys=[ns], tau_p=tau)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.empty(S, hq, d, device="cuda")
    gl, ge = torch.empty(hq, S, device="cuda"), torch.empty(1, hq, F, device="cuda")
    ws = torch.empty(ev.sparse_prefill_workspace(mask, d, cues=cues),
                     dtype=torch.uint8, device="cuda")
    more = {}
    if cues:
        n = mask.stats["n_frame_pairs"]
        more = {"frame_pairs": torch.empty(1, n, device="cuda"),
                "intra_frame": torch.empty(1, F, nv, nv, device="cuda")}
    ev.sparse_prefill(mask, 0, 1, cu(q), cu(k), cu(v), out, ge, ws, lse=gl,
                      **more)
    torch.cuda.synchronize()
    res = (out.cpu().numpy().astype(np.float64), gl.cpu().numpy(),
           ge[0].cpu().numpy())
    if cues:
        A = np.zeros((F, F))
        pr = ev.mask_export_pairs(mask)
        A[pr["a"], pr["b"]] = more["frame_pairs"][0].cpu().numpy()
        return res + (A, more["intra_frame"][0].cpu().numpy())
    return res


def _draw(S, hq, hkv, d, seed=5):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((S, h, d)).astype(np.float32)
            for h in (hq, hkv, hkv))


# Powers of two on Q, K and V: a value's three bf16 parts hold all its bits
# only while the lowest one is in bf16's range.
SCALES = {"small_v": (0, 0, -119), "least_v": (0, 0, -124),
          "small_q_large_k": (-122, 122, 0), "small_k_large_q": (122, -122, 0),
          "large_v": (0, 0, 108)}


@pytest.mark.parametrize("name", list(SCALES))
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_split_magnitudes(d, name):
    """Powers of two on the inputs change no relative error."""
    ns, F, nv, nt = 33, 4, 64, 32
    q, k, v = _draw(ns + F * nv + nt, 3, 1, d)
    # no value below fp32's normal range after the scale
    q, k, v = (np.copysign(np.maximum(np.abs(a), 2.0 ** -2), a).astype(
        np.float32) for a in (q, k, v))
    q, k, v = (np.ldexp(a, e) for a, e in zip((q, k, v), SCALES[name]))
    O, lse, E, _ = _reference(*(a.astype(np.float64) for a in (q, k, v)), ns,
                           ns + F * nv)
    out, gl, ge = _run(q, k, v, F, nv, nt, ns)
    # as below, and up to half of the least fp32 value, 2^-150, per output
    tiny = 2.0 ** -149 if SCALES[name][2] < 0 else 0.0
    assert np.abs(out - O).max() <= 1e-5 * np.abs(O).max() + tiny
    assert np.abs(gl - lse).max() <= 1e-5
    assert np.abs(ge - E.reshape(3, F, nv).sum(-1)).max() <= 1e-5 * nt


def test_fp32_split_small_probabilities():
    """A key 2^-123.6 of its row's largest whose value is 2^124 times the
    others' still counts in full."""
    d, n = 64, 64
    q, k, v = np.zeros((n + 1, 1, d), np.float32), np.zeros(
        (n + 1, 1, d), np.float32), np.ones((n + 1, 1, d), np.float32)
    q[:, 0, 0] = 8.0
    gap = np.float32(123.6 * np.log(2))          # logit of the other keys
    k[:, 0, 0], k[7, 0, 0] = gap, 0.0
    v[7] = np.ldexp(np.float32(1.37), 124)
    v[:, :, 1::2] = 0.0
    v[7, :, 1::2] = np.ldexp(np.float32(1.37), 124)
    O, _, _, _ = _reference(*(a.astype(np.float64) for a in (q, k, v)), 0, n)
    out, _, _ = _run(q, k, v, 1, n, 1, 0)
    # the probability's exponent, 123.6, is held to 2^-17 (two roundings)
    assert np.abs(out[8:] / O[8:] - 1).max() <= 2e-5


@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [(0, 3, 8, 1), (31, 5, 8, 33), (33, 4, 64, 32),
                                   (64, 3, 32, 65)])
def test_fp32_split(shape, d, infinite):
    ns, F, nv, nt = shape
    hq, hkv = 3, 1
    S = ns + F * nv + nt
    q, k, v = _draw(S, hq, hkv, d)
    skip = None
    if infinite:
        skip = ns + 2                       # a visual key, not its row's first
        q[:, :, 0] = -1.0 - np.abs(q[:, :, 0])
        k[skip, :, 0] = np.inf
    kr = np.where(np.isfinite(k), k, 0.0).astype(np.float64)
    O, lse, E, _ = _reference(q.astype(np.float64), kr, v.astype(np.float64), ns,
                           ns + F * nv, skip)
    out, gl, ge = _run(q, k, v, F, nv, nt, ns)
    # fp32 accumulation of d products per logit (|logit| < 16) and of up to S
    # probabilities, a few ulps each: 1e-5 covers both with a margin of ten
    assert np.abs(out - O).max() <= 1e-5 * np.abs(O).max()
    assert np.abs(gl - lse).max() <= 1e-5
    Ef = E.reshape(hq, F, nv).sum(-1)
    assert np.abs(ge - Ef).max() <= 1e-5 * max(nt, 1)


def _check(got, ref, hq, F, nv, nt, vis0, rows=slice(None)):
    out, gl, ge = got[:3]
    O, lse, E, p = ref
    # as above
    assert np.abs(out - O)[rows].max() <= 1e-5 * np.abs(O[rows]).max()
    assert np.abs(gl - lse).max() <= 1e-5
    assert np.abs(ge - E.reshape(hq, F, nv).sum(-1)).max() <= 1e-5 * nt
    if len(got) > 3:
        vis = p[:, vis0:vis0 + F * nv, vis0:vis0 + F * nv].mean(0)
        cell = vis.reshape(F, nv, F, nv)
        A = np.tril(cell.sum(3).mean(1), -1)
        own = cell[np.arange(F), :, np.arange(F)]
        assert np.abs(got[3] - A).max() <= 1e-5
        assert np.abs(got[4] - own).max() <= 1e-5


def _infinite_key(q, k, at):
    """Key ``at`` infinite in one component that gives it the logit -inf."""
    q[:, :, 0] = -1.0 - np.abs(q[:, :, 0])
    k[at, :, 0] = np.inf
    return np.where(np.isfinite(k), k, 0.0).astype(np.float64)


# items of 66 to 70 key tiles (paired ones too: three heads per kv head): the
# tiles' descriptors come 64 at a time
@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_split_many_tiles(d, infinite):
    ns, F, nv, nt, hq = 70, 68, 64, 40, 3
    S = ns + F * nv + nt
    q, k, v = _draw(S, hq, 1, d)
    at = ns + 65 * 64 + 9 if infinite else None     # in a row's 68th tile
    kr = _infinite_key(q, k, at) if infinite else k.astype(np.float64)
    ref = _reference(q.astype(np.float64), kr, v.astype(np.float64), ns,
                     ns + F * nv, at)
    _check(_run(q, k, v, F, nv, nt, ns), ref, hq, F, nv, nt, ns)


@pytest.mark.parametrize("tau", [0.0, 1.0])
@pytest.mark.parametrize("cues", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_split_infinite_key_forms(d, cues, tau):
    """tau = 1 keeps every block of positive probability: not the one with the
    infinite key, whose mean key has the affinity -inf."""
    ns, F, nv, nt, hq = 33, 9, 32, 40, 3
    S = ns + F * nv + nt
    q, k, v = _draw(S, hq, 1, d)
    at = ns + 70                                    # the second visual block
    kr = _infinite_key(q, k, at)
    drop = None
    if tau:
        rows = np.arange(S)
        drop = ((rows[:, None] >= ns + 128) & (rows[None] >= ns + 64) &
                (rows[None] < ns + 128))
    ref = _reference(q.astype(np.float64), kr, v.astype(np.float64), ns,
                     ns + F * nv, at, drop)
    got = _run(q, k, v, F, nv, nt, ns, tau, cues)
    _check(got, ref, hq, F, nv, nt, ns)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_split_infinite_value(d):
    """An infinite component of V is infinite in the rows of later blocks, whose
    other components, LSE and evidence are as ever."""
    ns, F, nv, nt, hq = 33, 5, 64, 40, 3
    S = ns + F * nv + nt
    q, k, v = _draw(S, hq, 1, d)
    at = ns + 64 + 11
    vr = v.astype(np.float64)
    v[at, 0, 7] = -np.inf
    ref = _reference(q.astype(np.float64), k.astype(np.float64), vr, ns,
                     ns + F * nv)
    out, gl, ge = _run(q, k, v, F, nv, nt, ns)
    assert (out[ns + 128:, :, 7] == -np.inf).all()
    keep = np.r_[0:ns + 64, ns + 128:S]             # not the key's own block
    out[:, :, 7] = ref[0][:, :, 7]
    _check((out, gl, ge), ref, hq, F, nv, nt, ns, keep)
