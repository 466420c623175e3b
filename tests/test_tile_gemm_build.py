"""Build-time guard of the any-width grouped GEMMs: their weights are loaded into registers by inline asm that the
compiler does not track and read only after an explicit wait (and so are the token fragments, from LDS), so the
kernels must neither spill nor use scratch, and no instruction may touch such a register between its load and the
marker after the wait."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_21868_amd import build


def _regs(s):
    out = set()
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", s):
        out |= set(range(int(a), int(b) + 1))
    return out | {int(a) for a in re.findall(r"\bv(\d+)\b", s)}


@pytest.mark.skipif(not (shutil.which(build.HIPCC) or os.path.exists(build.HIPCC)), reason="hipcc not installed")
def test_tile_kernels_keep_their_registers(tmp_path):
    asm = tmp_path / "t.s"
    r = subprocess.run([build.HIPCC, *build.HIP_FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "tile_gemm.hip"),
                        "-o", str(asm)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:]
    seen = 0
    for part in re.split(r"\n(?=_ZN4wisp\S+:)", asm.read_text())[1:]:
        name = part.split(":")[0]
        if "tile_kernel" not in name:
            continue
        seen += 1
        assert re.search(r"; ScratchSize: 0\b", part) and int(re.search(r"; NumVgprs: (\d+)", part).group(1)) <= 256, name
        lines = [l.strip() for l in part.split(".Lfunc_end")[0].split("\n")]
        labels = {l.split(":")[0]: i for i, l in enumerate(lines) if re.match(r"\.LBB\S+:", l)}
        # the main loop: the longest branch back.  Its body is gone through again with what the pass before left in flight (the
        # pair order is loaded a whole tile ahead and pinned in a later turn)
        jumps = [(i, labels.get(m.group(1), i)) for i, l in enumerate(lines) if (m := re.match(r"s_c?branch\S* (\.LBB\S+)", l))]
        end, start = max(jumps, key=lambda j: j[0] - j[1])
        assert end - start > len(lines) // 2, name
        in_flight, loads, pairs = set(), 0, 0
        for s in lines + lines[start:]:
            if s.startswith("; pin"):
                in_flight -= _regs(s)
                continue
            if not s or s[0] in ";.":
                continue
            m = re.match(r"(buffer_load_dwordx4|buffer_load_ushort|global_load_dword|ds_read_b128) (v\[\d+:\d+\]|v\d+), ", s)
            if m and not s.endswith("lds"):
                loads += 1
                pairs += m.group(1) == "global_load_dword"
                assert not _regs(s[m.end():]) & in_flight, (name, s)
                assert m.group(1) != "global_load_dword" or not _regs(m.group(2)) & in_flight, (name, s)
                in_flight |= _regs(m.group(2))
            else:
                assert not _regs(s) & in_flight, (name, s)
        assert pairs >= 8, name
        assert loads >= 16, name
    assert seen == 8
