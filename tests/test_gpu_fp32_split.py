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


@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", [(0, 3, 8, 1), (31, 5, 8, 33), (33, 4, 64, 32),
                                   (64, 3, 32, 65)])
def test_fp32_split(shape, d, infinite):
    import torch
    ev = pytest.ev
    ns, F, nv, nt = shape
    hq, hkv = 3, 1
    S = ns + F * nv + nt
    rng = np.random.default_rng(5)
    q, k, v = (rng.standard_normal((S, h, d)).astype(np.float32)
               for h in (hq, hkv, hkv))
    skip = None
    if infinite:
        skip = ns + 2                       # a visual key, not its row's first
        q[:, :, 0] = -1.0 - np.abs(q[:, :, 0])
        k[skip, :, 0] = np.inf
    kr = np.where(np.isfinite(k), k, 0.0).astype(np.float64)
    O, lse, E = _reference(q.astype(np.float64), kr, v.astype(np.float64), ns,
                           ns + F * nv, skip)
    mask = ev.build_block_mask([F], [nt], nv, 64, 1, -1, hq, hkv, n_sys=[ns])
    cu = lambda a: torch.from_numpy(a).cuda()
    out = torch.empty(S, hq, d, device="cuda")
    gl, ge = torch.empty(hq, S, device="cuda"), torch.empty(1, hq, F, device="cuda")
    ws = torch.empty(ev.sparse_prefill_workspace(mask, d), dtype=torch.uint8,
                     device="cuda")
    ev.sparse_prefill(mask, 0, 1, cu(q), cu(k), cu(v), out, ge, ws, lse=gl)
    torch.cuda.synchronize()
    # fp32 accumulation of d products per logit (|logit| < 16) and of up to S
    # probabilities, a few ulps each: 1e-5 covers both with a margin of ten
    assert np.abs(out.cpu().numpy() - O).max() <= 1e-5 * np.abs(O).max()
    assert np.abs(gl.cpu().numpy() - lse).max() <= 1e-5
    Ef = E.reshape(hq, F, nv).sum(-1)
    assert np.abs(ge[0].cpu().numpy() - Ef).max() <= 1e-5 * max(nt, 1)
