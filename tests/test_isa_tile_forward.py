"""The build-time guard of test_isa_guards.py for the activation reads of tile_fwd_kernel (no GPU needed)."""
import os
import re
import subprocess

from paper_2210_03858_amd import build
from test_isa_guards import ROOT, _check


def test_no_tile_forward_touches_a_fragment_before_its_wait(tmp_path):
    src, out = os.path.join(ROOT, "paper_2210_03858_amd", "csrc", "bcq_fused.hip"), str(tmp_path / "bcq_fused.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    r = subprocess.run([build._hipcc()] + flags + ["-S", "--cuda-device-only", src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    bodies = re.findall(r"^(_ZN3bcq15tile_fwd_kernelILi\dELi\dELi\dELb\dEE\w*):[^\n]*\n(.*?)\.Lfunc_end", open(out).read(), re.S | re.M)
    assert len(bodies) == 16  # one to four planes, two tiles, row- and group-wise scales
    for name, body in bodies:
        lines = [l.strip() for l in body.split("\n")]
        lines = [l for l in lines if l and l[0] not in ";."]
        reads, violations = _check(lines)
        tokens = int(re.search(r"kernelILi\dELi(\d)", name).group(1))
        assert reads >= 8 * tokens and not violations, (name, reads, violations[:5])  # two units, four slices, a read for 16 tokens
        assert not any("scratch_" in l for l in lines), name
