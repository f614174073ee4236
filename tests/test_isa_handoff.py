"""What the workgroups of one Gauss-Newton sample hand each other (CPU only: reads
the gfx950 assembly that hipcc writes for this library's own kernels).

Partial sums and estimates are stored past the XCD's cache (device-scope atomic
stores, `sc1`) and announced by a counter, with no fence in between: each such
store must have completed (`s_waitcnt` with vmcnt(0)) before the workgroup's next
barrier, behind which one thread changes the counter.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_07759_amd", "csrc")
HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")


def unfinished(lines):
    """(stores handed on, lines of those that reach a barrier unfinished)."""
    n, bad = 0, []
    for i, l in enumerate(lines):
        if not re.match(r"\s*global_store_dwordx2 .*\bsc1\b", l):
            continue
        n += 1
        for later in lines[i + 1:]:
            s = later.strip()
            if re.match(r"s_waitcnt\b.*vmcnt\(0\)", s):
                break
            if s.startswith("s_barrier") or s.startswith("s_endpgm"):
                bad.append(i + 1)
                break
    return n, bad


def kernels(asm_text, name):
    """Lines of each function whose (mangled) name holds `name`."""
    out, cur = {}, None
    for l in asm_text.split("\n"):
        m = re.match(r"^(_Z\w+):", l)
        if m:
            cur = out.setdefault(m.group(1), []) if name in m.group(1) else None
        elif cur is not None:
            cur.append(l)
    return out


def test_scan_finds_a_store_in_flight():
    store = "  global_store_dwordx2 v[2:3], v[0:1], off sc1"
    assert unfinished([store, "  s_waitcnt lgkmcnt(0)", "  s_barrier"]) == (1, [1])
    assert unfinished([store, "  s_waitcnt vmcnt(0)", "  s_barrier"]) == (1, [])


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_sums_and_estimates_land_before_they_are_announced(tmp_path):
    out = str(tmp_path / "im_build.s")
    r = subprocess.run(
        [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++20", "-Xclang", "-target-feature",
         "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-x", "hip", "-S",
         "--cuda-device-only", os.path.join(CSRC, "im_build.hip"), "-o", out],
        capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = kernels(open(out).read(), "gn_lds_kernelILb1")   # several workgroups a sample
    assert len(found) == 3
    for name, lines in found.items():
        n, bad = unfinished(lines)
        assert n == 2 and not bad, (name, n, bad)   # a workgroup's sums, the new estimate
