"""Code generation of the grouped GEMMs (CPU only: hipcc cross-compiles gfx950 device assembly).

Some tile configurations use all 256 architectural registers of a wave and spill a few values
to scratch.  Those accesses must stay outside the K loops: inside, a scratch load is a vector
memory load like the slice copies, and waiting for it (vmcnt counts in issue order) would also
wait for every copy in flight.  For every kernel with MFMAs this test finds its innermost loops
that contain MFMAs (a backward branch to an earlier label) and checks that no scratch access sits
inside one.

The slice copies written as inline assembly keep the wait state between a scalar write of M0 (their
LDS address) and the direct-to-LDS load that reads it, which the compiler does not see."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_18631_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")


def _device_asm(src, out):
    from paper_2607_18631_amd import build
    cmd = [HIPCC, *build.FLAGS, "-I", CSRC, "-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    with open(out) as f:
        return f.read()


def _mfma_loops(lines):
    """(first, last) line spans of the innermost loops that contain an MFMA."""
    labels = {}
    for i, l in enumerate(lines):
        m = re.match(r"(\.LBB\d+_\d+):", l)
        if m:
            labels[m.group(1)] = i
    loops = []
    for i, l in enumerate(lines):
        m = re.search(r"s_(?:cbranch_\w+|branch)\s+(\.LBB\d+_\d+)", l)
        if m and m.group(1) in labels and labels[m.group(1)] < i:
            loops.append((labels[m.group(1)], i))
    has_mfma = [(a, b) for a, b in loops if any("v_mfma" in lines[k] for k in range(a, b))]
    return [(a, b) for a, b in has_mfma
            if not any((c, d) != (a, b) and a <= c and d <= b for c, d in has_mfma)]


@pytest.fixture(scope="module")
def device_asm(tmp_path_factory):
    d = tmp_path_factory.mktemp("asm")
    srcs = ["gemm.hip", "gemm_phase.hip", "gemm_bwd.hip"]
    with ThreadPoolExecutor(len(srcs)) as ex:
        texts = list(ex.map(lambda s: _device_asm(s, str(d / (s + ".s"))), srcs))
    return dict(zip(srcs, texts))


def _tile_code(lines):
    """Code of the tile loop: an epilogue's stores, or the accumulators' zeroing."""
    return any("global_store" in l for l in lines) or sum(bool(re.search(r"v_mov_b(32|64)\S* v(\d+|\[\d+:\d+\]), ", l)) for l in lines) > 16


@pytest.mark.parametrize("src", ["gemm.hip", "gemm_phase.hip", "gemm_bwd.hip"])
def test_no_scratch_in_mfma_loops(device_asm, src):
    funcs = re.split(r"\n(?=_Z\S+:)", device_asm[src])
    checked = 0
    for f in funcs:
        if "v_mfma" not in f:
            continue
        name = f.split(":", 1)[0]
        lines = f.split("\n")
        loops = _mfma_loops(lines)
        if src == "gemm_phase.hip":
            # one K loop per count of phases and live blocks; the code around them (the last slices of each) is
            # laid out with backward branches too
            loops = [(a, b) for a, b in loops if not _tile_code(lines[a:b + 1])]
        assert loops, f"no MFMA loop found in {name}"
        inside = [lines[i].strip() for a, b in loops for i in range(a, b + 1) if "scratch_" in lines[i]]
        assert not inside, f"{name}: scratch accesses inside an MFMA loop: {inside[:4]}"
        checked += 1
    assert checked >= 8, f"only {checked} MFMA kernels found in {src}"
    print(f"[codegen] {src}: {checked} MFMA kernels, no scratch access inside their K loops")


def _reloads_between_mfmas(lines, near=30):
    """Scratch loads with an MFMA within `near` instructions on both sides."""
    ins = [l.split(";")[0].strip() for l in lines]
    ins = [l for l in ins if l and not l.startswith(".") and not l.endswith(":")]
    mfma = [i for i, l in enumerate(ins) if l.startswith("v_mfma")]
    close = lambda i: any(0 < i - m <= near for m in mfma) and any(0 < m - i <= near for m in mfma)
    return sum(l.startswith("scratch_load") and close(i) for i, l in enumerate(ins))


@pytest.mark.parametrize("src", ["gemm_phase.hip", "gemm_bwd.hip"])
def test_few_reloads_between_mfmas(device_asm, src):
    """A reload between MFMAs waits for the copies in flight, in a tile's last slices as well as in its K loop.  At most
    the four fragment offsets, once per tile, behind the K loop."""
    checked = 0
    for f in re.split(r"\n(?=_Z\S+:)", device_asm[src]):
        if "v_mfma" in f and "k_phase" in f.split(":", 1)[0]:
            n = _reloads_between_mfmas(f.split("\n"))
            assert n <= 4, f"{f.split(':', 1)[0]}: {n} reloads between MFMAs"
            checked += 1
    assert checked >= 4


def test_reload_finder():
    m, load = "\tv_mfma_f32_16x16x32_bf16 v[0:3]", "\tscratch_load_dword v3, off, off offset:36 ; 4-byte Folded Reload"
    far = ["\tv_mov_b32_e32 v1, v2"] * 40
    assert _reloads_between_mfmas([m, load, "\ts_waitcnt vmcnt(0)", m]) == 1
    assert _reloads_between_mfmas([m, load, *far, m]) == 0 and _reloads_between_mfmas([m, *far, load, m]) == 0


def test_weight_gradients_are_stored_nontemporally(device_asm):
    """The results of the large-tile weight-gradient kernel, and an empty group's zeros where rows are whole lines: they
    are written once and not read again by the step, and must not displace its weights in the last-level cache.
    Only the zeros of other rows (one loop of four stores) are temporal."""
    f = [f for f in re.split(r"\n(?=_Z\S+:)", device_asm["gemm_bwd.hip"])
         if "k_phase_bwdILi256ELi1E" in f.split(":", 1)[0] and "v_mfma" in f]
    assert len(f) == 1
    stores = [bool(re.search(r"\bnt\b", l)) for l in f[0].split("\n") if "global_store_dwordx4" in l]
    assert sum(stores) >= 16 + 4 and len(stores) - sum(stores) <= 4, stores


def _m0_hazards(lines):
    """Direct-to-LDS loads whose very next preceding instruction writes M0 by a scalar instruction."""
    found, prev = [], ""
    for l in lines:
        ins = l.split(";")[0].strip()
        if not ins or ins.endswith(":") or ins.startswith("."):
            continue
        if re.match(r"(global|buffer|scratch)_load_lds|buffer_load_\w+ .*\blds\b", ins) and re.match(r"s_\w+\s+m0\b", prev):
            found.append((prev, ins))
        prev = ins
    return found


@pytest.mark.parametrize("src", ["gemm.hip", "gemm_phase.hip", "gemm_bwd.hip"])
def test_lds_copies_wait_for_m0(device_asm, src):
    lines = device_asm[src].split("\n")
    copies = sum("global_load_lds" in l for l in lines)
    assert copies >= 100, f"only {copies} slice copies found in {src}"
    bad = _m0_hazards(lines)
    assert not bad, f"{len(bad)} of {copies} copies directly behind a write of M0: {bad[:2]}"


def test_m0_finder():
    """On hand-written listings: a copy right behind a write of M0 (assembler comments and a label
    between) is found; one with a wait state, another instruction or another register is not."""
    bad = "\ts_mov_b32 m0, s1\n\t;;#x\n.Lcopy0:\n\tglobal_load_lds_dwordx4 v1, s[2:3]"
    assert len(_m0_hazards(bad.split("\n"))) == 1
    for mid in ("\ts_nop 0\n", "\ts_cmp_eq_u32 s4, 0\n", "\ts_mov_b32 s5, s6\n"):
        assert not _m0_hazards(("\ts_mov_b32 m0, s1\n" + mid + "\tglobal_load_lds_dwordx4 v1, s[2:3]").split("\n"))


def test_loop_finder_sees_scratch_in_a_loop():
    """The loop finder on a hand-written listing: a scratch reload inside the MFMA loop is found,
    one in the prologue or in an outer loop's tile code is not."""
    asm = """_Zk:
\tscratch_load_dword v1, off, off
.LBB0_1:
\tscratch_load_dword v2, off, off offset:4
.LBB0_2:
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]
\tscratch_load_dword v3, off, off offset:8
\ts_cbranch_scc1 .LBB0_2
\tglobal_store_dword v0, v1, s[0:1]
\ts_cbranch_vccnz .LBB0_1
\ts_endpgm""".split("\n")
    loops = _mfma_loops(asm)
    assert loops == [(4, 7)]
    inside = [asm[i] for a, b in loops for i in range(a, b + 1) if "scratch_" in asm[i]]
    assert inside == ["\tscratch_load_dword v3, off, off offset:8"]
