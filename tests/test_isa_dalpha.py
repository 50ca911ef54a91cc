"""The build-time guard of test_isa_guards.py for the transposing fragment reads of dalpha_kernel (no GPU needed)."""
import re

from test_isa_guards import _check, mfma_asm  # noqa: F401  (mfma_asm: fixture)


def test_no_dalpha_kernel_touches_a_fragment_before_its_wait(mfma_asm):  # noqa: F811
    bodies = re.findall(r"^(_ZN3bcq13dalpha_kernelILi\d+ELi\d+ELb\dEE\w*):[^\n]*\n(.*?)s_endpgm", mfma_asm, re.S | re.M)
    assert len(bodies) == 20  # two tiles, five plane counts, row- and group-wise partial sums
    for name, body in bodies:
        lines = [l.strip() for l in body.split("\n")]
        lines = [l.replace("ds_read_b64_tr_b16", "ds_read_b128") for l in lines if l and l[0] not in ";."]
        reads, violations = _check(lines)
        assert reads >= 48 and not violations, (name, reads, violations[:5])
        assert not any("scratch_" in l for l in lines), name
