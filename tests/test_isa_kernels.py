"""Static checks of the built step kernels beside those of test_isa_order: what
the registers leave to each kernel, and the order and arithmetic of the kernels
that boxes run by default."""
import re

from test_isa_order import asm  # noqa: F401  (the module's fixture)


def _metadata(asm, pattern):  # noqa: F811
    """{kernel: {.vgpr_count: ..., ...}} from the code object metadata."""
    out = {}
    for block in re.split(r"\n  - \.agpr_count:", asm)[1:]:
        block = ".agpr_count:" + block
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        if re.search(pattern, name):
            out[name] = {k: int(v) for k, v in re.findall(r"(\.\w+):\s+(\d+)\n", block)}
    return out


def test_exact_stabilizer_statistics_fit_two_waves_per_simd(asm):  # noqa: F811
    """512 registers per lane and SIMD, 160 KB of LDS per CU: at most 256 registers
    and 80 KB per four-wave workgroup."""
    ks = _metadata(asm, r"k_gamma_statsILi\dELi\dELb1E")
    assert len(ks) == 4 * 8
    for nm, m in ks.items():
        assert m[".vgpr_count"] <= 256, (nm, m[".vgpr_count"])
        assert m[".group_segment_fixed_size"] <= 80 * 1024, nm
