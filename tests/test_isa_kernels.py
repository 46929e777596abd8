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


def test_exact_pull_sweeps_issue_their_loads_together(asm):  # noqa: F811
    """27 population loads with no wait between them in FP16, where the scheduler
    had placed one after each, and at most two in the other forms (it holds
    the last few back): a wait is a whole memory latency for every node."""
    names = re.findall(r"^(_ZN3kbc\S*k_stepILi\dELi\dELi0ELb1\S*):", asm, flags=re.M)
    # 4 storage forms x 8 variants x (generic, 64-node chunks)
    assert len(names) == 4 * 8 * 2
    for nm in names:
        i = asm.index(nm + ":")
        lines = [ln.strip() for ln in asm[i:asm.index(".Lfunc_end", i)].split("\n")]
        loads = [k for k, ln in enumerate(lines) if ln.startswith("global_load")]
        assert len(loads) == 27, (nm, len(loads))
        waits = [ln for ln in lines[:loads[-1]] if ln.startswith("s_waitcnt") and "vmcnt" in ln]
        assert len(waits) <= (0 if "k_stepILi2E" in nm else 2), (nm, len(waits))
