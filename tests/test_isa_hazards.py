"""Compiled-code check of the direct global -> LDS loads (CPU only: hipcc
cross-compiles the attention sources for gfx950 to assembly).

On gfx9 a vector-memory instruction that reads an SGPR written by a VALU
instruction needs five wait states in between. The compiler inserts them
for the memory instructions it emits itself, but the tile loads are inline
assembly (global_load_lds_dwordx4 with a scalar base), whose operands the
compiler may fill from spilled SGPRs with v_readlane_b32 right before the
instruction. Without the wait states the load can take a stale base and
address arbitrary memory. The loads therefore start with their own
s_nop 4; this test scans every kernel of the attention sources and fails
on any load whose SGPR base, or m0, was written by a VALU instruction fewer
than five wait states earlier, or whose base is not in SGPRs at all.

The same compile, of the retention and coarse sources too, reports each
kernel's registers: none may spill VGPRs (to scratch memory) past the counts
recorded here, and the SGPR spills (to VGPR lanes, a v_writelane / v_readlane
pair each) of the attention and coarse kernels may not grow past theirs."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_05780_amd", "csrc")
SOURCES = ["attn.hip", "attn_pipe.hip"]
SPILL_SOURCES = SOURCES + ["select.hip", "evidence.hip"]
WAIT_STATES = 5
# SGPR spills per kernel at the current sources (kernel name fragment ->
# spills); none of the pipelined kernel's is reloaded inside its tile loop
SGPR_SPILL_BUDGET = {
    "attn_pipe_kernelILi128ELb0": 86, "attn_pipe_kernelILi64ELb0": 82,
    # the pipelined kernel's frame-cue form (tile CSR positions in the
    # descriptors, visual-row partials and LSE)
    "attn_pipe_kernelILi128ELb1": 76, "attn_pipe_kernelILi64ELb1": 81,
    # its top-p form (retention bits, candidate list)
    "attn_pipe_topp_kernelILi128": 119, "attn_pipe_topp_kernelILi64": 110,
    "attn_kernelINS0_8Bf16PathILi128EEELi128ELb0": 93,
    "attn_kernelINS0_8Bf16PathILi128EEELi128ELb1": 104,
    "attn_kernelINS0_8Bf16PathILi64EEELi64ELb0": 92,
    "attn_kernelINS0_8Bf16PathILi64EEELi64ELb1": 98,
    "attn_kernelINS0_7F32PathILi128EEELi128ELb0": 54,
    "attn_kernelINS0_7F32PathILi128EEELi128ELb1": 67,
    "attn_kernelINS0_7F32PathILi64EEELi64ELb0": 44,
    "attn_kernelINS0_7F32PathILi64EEELi64ELb1": 65,
    # the intra-frame kernel stages each head pair's query rows with the
    # tile loader (bf16), which holds the loader's offsets across the loop
    "intra_kernelINS0_8Bf16PathILi128": 74, "intra_kernelINS0_8Bf16PathILi64": 74,
    "intra_kernelINS0_7F32PathILi128": 0, "intra_kernelINS0_7F32PathILi64": 0,
    "coarse_kernel": 0,
}
# VGPR spills (lanes to scratch memory) that are allowed: one register of the
# selection, the price of four waves per SIMD
VGPR_SPILL_BUDGET = {"select_kernel": 1}


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc",
              shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    return None


def _sregs(tok):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", tok)
    if m:
        return {f"s{i}" for i in range(int(m.group(1)), int(m.group(2)) + 1)}
    m = re.fullmatch(r"s(\d+)", tok)
    if m:
        return {tok}
    if tok in ("vcc", "vcc_lo", "vcc_hi", "m0"):
        return {"vcc_lo", "vcc_hi"} if tok == "vcc" else {tok}
    return set()


def _valu_sgpr_defs(ins):
    """SGPRs (and m0) a VALU instruction writes."""
    op, *args = ins.replace(",", " ").split()
    if not op.startswith("v_"):
        return set()
    out = set()
    if op.startswith(("v_readlane", "v_readfirstlane")):
        out |= _sregs(args[0])
    elif op.startswith("v_cmp") and op.endswith("_e64"):
        out |= _sregs(args[0])
    elif op.startswith("v_cmp"):
        out |= {"vcc_lo", "vcc_hi"}
    elif ("_co_" in op or op.startswith(("v_mad_u64", "v_mad_i64",
                                         "v_div_scale"))) and len(args) > 1:
        out |= _sregs(args[1])
    return out


def scan(asm_text):
    """(number of LDS-DMA loads, list of violations) of one .s file."""
    n, bad = 0, []
    hist = []   # (wait states, SGPRs written by VALU, text)
    fn = "?"
    for line in asm_text.split("\n"):
        t = line.strip()
        m = re.match(r"^(_Z\w+):", t)
        if m:
            fn, hist = m.group(1), []
            continue
        if not t or t.startswith((";", ".")) or t.endswith(":"):
            continue
        if t.startswith("global_load_lds"):
            n += 1
            base = t.replace(",", " ").split()[2]
            uses = _sregs(base)
            if not uses:
                bad.append((fn, t, "base not in SGPRs"))
            uses = uses | {"m0"}
            ws = 0
            for w, defs, txt in reversed(hist):
                if ws >= WAIT_STATES:
                    break
                if defs & uses:
                    bad.append((fn, t, f"{ws} wait states after {txt}"))
                    break
                ws += w
        op = t.split()[0]
        w = int(t.split()[1], 0) + 1 if op == "s_nop" else 1
        hist.append((w, _valu_sgpr_defs(t), t))
        hist = hist[-16:]
    return n, bad


def test_scanner_flags_the_hazard():
    """The scanner itself: a load right after a spill reload is flagged,
    the same load behind s_nop 4 is not."""
    hazard = """_Zk:
\tv_readlane_b32 s7, v227, 54
\ts_mov_b32 m0, s33
\ts_nop 0
\tglobal_load_lds_dwordx4 v2, s[6:7]
"""
    n, bad = scan(hazard)
    assert n == 1 and len(bad) == 1
    n, bad = scan(hazard.replace("s_nop 0", "s_nop 4"))
    assert n == 1 and not bad
    n, bad = scan(hazard.replace("s[6:7]", "v[6:7]"))
    assert bad and "SGPR" in bad[0][2]


@pytest.mark.slow
def test_lds_dma_operands_have_their_wait_states(tmp_path):
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not available")

    def compile_one(src):
        out = tmp_path / (src + ".s")
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-I", os.path.join(ROOT, "include"), "-I", CSRC,
               "--cuda-device-only", "-S", os.path.join(CSRC, src),
               "-o", str(out), "-Rpass-analysis=kernel-resource-usage"]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return out.read_text(), r.stderr

    with ThreadPoolExecutor(len(SPILL_SOURCES)) as ex:
        results = list(ex.map(compile_one, SPILL_SOURCES))
    texts = [t for t, _ in results[:len(SOURCES)]]
    usage = {}
    for _, remarks in results:
        name = None
        for line in remarks.splitlines():
            m = re.search(r"Function Name: (\S+)", line)
            if m:
                name = m.group(1)
            m = re.search(r"(SGPRs|VGPRs) Spill: (\d+)", line)
            if m and name:
                usage.setdefault(name, {})[m.group(1)] = int(m.group(2))
    seen = set()
    for name, u in usage.items():
        vgprs = [n for frag, n in VGPR_SPILL_BUDGET.items() if frag in name]
        assert u["VGPRs"] <= sum(vgprs), (name, u)
        frags = [frag for frag in SGPR_SPILL_BUDGET if frag in name]
        if "attn" in name or "intra" in name or "coarse_kernel" in name:
            assert len(frags) == 1, (name, frags)
            assert u["SGPRs"] <= SGPR_SPILL_BUDGET[frags[0]], (name, u)
            seen.update(frags)
    assert seen == set(SGPR_SPILL_BUDGET), set(SGPR_SPILL_BUDGET) - seen
    total = 0
    for src, text in zip(SOURCES, texts):
        n, bad = scan(text)
        total += n
        assert not bad, (src, bad[:5])
    assert total > 500   # every attention kernel variant was scanned
