"""Hand-written global-to-LDS loads in the compiled kernels (CPU only: reads the gfx950 assembly of the sources here).

Such a load takes its LDS address from m0 and needs one wait state after the scalar write of m0; the compiler adds
it between its own instructions but not inside an asm block."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_08802_amd", "csrc")


def _sources():
    out = []
    for f in sorted(os.listdir(CSRC)):
        if f.endswith(".hip"):
            with open(os.path.join(CSRC, f)) as h:
                if re.search(r"load_lds|_load_dword.* lds", h.read()):
                    out.append(f)
    return out


def unwaited_loads(asm):
    """(loads to LDS, those issued right after a write of m0)"""
    n, bad, before = 0, [], ""
    for line in asm.splitlines():
        ins = line.split(";")[0].strip()
        if not ins or ins.startswith(".") or ins.endswith(":"):     # comments, directives, labels
            continue
        if re.match(r"(global|buffer)_load_lds_|buffer_load_\S+ .*\blds\b", ins):
            n += 1
            if re.match(r"s_\S+\s+m0\b", before):
                bad.append(f"{before} / {ins}")
        before = ins
    return n, bad


def test_detects_a_missing_wait():
    load = "\tglobal_load_lds_dwordx4 v1, s[2:3]\n"
    assert unwaited_loads("\ts_mov_b32 m0, s4\n\t;;#ASMSTART\n" + load)[1]
    assert unwaited_loads("\ts_mov_b32 m0, s4\n\ts_nop 0\n" + load) == (1, [])


@pytest.mark.parametrize("src", _sources())
def test_wait_state_after_m0(src, tmp_path):
    sys.path.insert(0, ROOT)
    import __graft_entry__ as G
    out = tmp_path / "k.s"
    r = subprocess.run(["hipcc"] + G.HIPCC_FLAGS + ["--offload-device-only", "-S", os.path.join(CSRC, src), "-o",
                                                    str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    n, bad = unwaited_loads(out.read_text())
    assert n > 0 and not bad, (n, bad[:3])
