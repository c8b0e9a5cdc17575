"""Top-p attention in the pipelined kernel against the plain one (which serves
the same call when frame cues are requested): frames of every length, paired
heads, short tails, query rows cut into chunks some of whose rows keep none of
the chunk's tiles, and logits that rise or fall far beyond a row's first
tile's (the pipelined kernel's recomputation). The same inputs go through the
pipelined kernel against the oracle too."""
import pytest

import workloads as wl
from gpu_harness import to_device
from test_gpu_topp import _run_case, _scale_queries

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    pytest.ev = gpu_lib


def _w(nv, d, hq, hkv, frames, text, ns, struct=(2.0, 2.0, 0.8)):
    return wl.Workload(
        name=f"topp-pipe-{nv}-{d}", config_id=903, n_layers=1, hq=hq, hkv=hkv,
        d=d, dtype="bf16", tokens_per_frame=nv, block=64, sink_blocks=1,
        window=8, plant="choose", n_frames=frames, n_text=text, n_sys=ns,
        n_videos=len(frames), tau_p=0.9, key_struct=struct,
        plant_args={"count": 2, "s_frame": (2.0, 3.0), "s_query": 2.0})


CASES = {
    "nv64_d128_odd": (_w(64, 128, 3, 1, (21,), (130,), (0,)), 1.0),
    "nv32_d64_sys": (_w(32, 64, 4, 2, (9, 31), (1, 70), (65, 3)), 1.0),
    "nv16_d128": (_w(16, 128, 2, 2, (50,), (40,), (7,)), 1.0),
    "nv8_d64_odd": (_w(8, 64, 3, 1, (77, 5), (66, 9), (0, 1)), 1.0),
    "far_logits": (_w(64, 128, 3, 1, (12,), (70,), (10,)), 60.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_pipelined_matches_plain(name):
    import torch
    ev = pytest.ev
    w, scale = CASES[name]
    ns, nf, nt = wl.layout_arrays(w)
    q, k, v = to_device(wl.gen_layer(w, 0), w, torch)
    q = (q.float() * scale).bfloat16()
    mask = ev.build_block_mask(nf, nt, w.tokens_per_frame, 64, 1, 8, w.hq,
                               w.hkv, n_sys=ns, tau_p=w.tau_p)
    st, nv = mask.stats, w.tokens_per_frame
    S, T = st["n_tokens"], st["n_frames_total"]
    ws = torch.empty(ev.sparse_prefill_workspace(mask, w.d, cues=True),
                     dtype=torch.uint8, device="cuda")
    res = []
    for cues in (False, True):
        f = lambda *s: torch.full(s, float("nan"), device="cuda")
        out = torch.zeros(S, w.hq, w.d, dtype=torch.bfloat16, device="cuda")
        lse, e, tm = f(w.hq, S), f(1, w.hq, T), f(1, w.hq, len(nf))
        more = {"frame_pairs": f(1, max(st["n_frame_pairs"], 1)),
                "intra_frame": f(1, T, nv, nv)} if cues else {}
        ev.sparse_prefill(mask, 0, 1, q, k, v, out, e, ws, lse=lse,
                          text_mass=tm, **more)
        torch.cuda.synchronize()
        res.append((out.float(), lse, e, tm))
    (oa, la, ea, ta), (ob, lb, eb, tb) = res
    # the same bf16 products; P is rounded at another scale (2^-9 of P) and O
    # once (2^-9); the sums are fp32 in another order
    assert (oa - ob).abs().max() <= 1e-2 * ob.abs().max()
    assert (la - lb).abs().max() <= 1e-5 * lb.abs().max()
    rows = max(int(x) for x in nt)
    assert (ea - eb).abs().max() <= 1e-5 * rows
    assert (ta - tb).abs().max() <= 1e-5 * rows


@pytest.mark.parametrize("name", list(CASES))
def test_pipelined_matches_oracle(name):
    w, scale = CASES[name]
    _run_case(w, transform=None if scale == 1.0 else
              lambda x, lay, blk: _scale_queries(x, lay, blk, scale))
