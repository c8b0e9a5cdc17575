"""The fp32 attention (three-way bf16 split) where its 32-key half tiles and
its fallback matter, against fp64: block lengths around the halves, both head
dims, and keys whose split is not finite (an infinite key component that gives
the key the logit -inf must leave the rows as if the key were not there)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    pytest.ev = gpu_lib


def _reference(q, k, v, vis0, txt0, skip=None):
    """Plain causal attention in fp64 (one video, window -1)."""
    S, hq, d = q.shape
    grp = hq // k.shape[1]
    k, v = np.repeat(k, grp, 1), np.repeat(v, grp, 1)
    s = np.einsum("ihd,jhd->hij", q, k) * d ** -0.5
    s[:, np.triu(np.ones((S, S), bool), 1)] = -np.inf
    if skip is not None:
        s[:, :, skip] = -np.inf
    m = s.max(-1, keepdims=True)
    p = np.exp(s - m)
    z = p.sum(-1, keepdims=True)
    p /= z
    E = p[:, txt0:, vis0:txt0].sum(1)
    return np.einsum("hij,jhd->ihd", p, v), (m + np.log(z))[..., 0], E


def _run(q, k, v, F, nv, nt, ns, tau=0.0):
    import torch
    ev = pytest.ev
    S, hq, d = q.shape
    mask = ev.build_block_mask([F], [nt], nv, 64, 1, -1, hq, k.shape[1],
                               n_sys=[ns], tau_p=tau)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.empty(S, hq, d, device="cuda")
    gl, ge = torch.empty(hq, S, device="cuda"), torch.empty(1, hq, F, device="cuda")
    ws = torch.empty(ev.sparse_prefill_workspace(mask, d), dtype=torch.uint8,
                     device="cuda")
    ev.sparse_prefill(mask, 0, 1, cu(q), cu(k), cu(v), out, ge, ws, lse=gl)
    torch.cuda.synchronize()
    return (out.cpu().numpy().astype(np.float64), gl.cpu().numpy(),
            ge[0].cpu().numpy())


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
    O, lse, E = _reference(*(a.astype(np.float64) for a in (q, k, v)), ns,
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
    O, _, _ = _reference(*(a.astype(np.float64) for a in (q, k, v)), 0, n)
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
    O, lse, E = _reference(q.astype(np.float64), kr, v.astype(np.float64), ns,
                           ns + F * nv, skip)
    out, gl, ge = _run(q, k, v, F, nv, nt, ns)
    # fp32 accumulation of d products per logit (|logit| < 16) and of up to S
    # probabilities, a few ulps each: 1e-5 covers both with a margin of ten
    assert np.abs(out - O).max() <= 1e-5 * np.abs(O).max()
    assert np.abs(gl - lse).max() <= 1e-5
    Ef = E.reshape(hq, F, nv).sum(-1)
    assert np.abs(ge - Ef).max() <= 1e-5 * max(nt, 1)
