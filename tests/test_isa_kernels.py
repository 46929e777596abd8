"""Static checks of the built step kernels beside those of test_isa_order: what
the registers leave to each kernel, and the order and arithmetic of the kernels
that boxes run by default."""
import re
from collections import Counter

from test_isa_order import _fp_ops, _kernels, asm  # noqa: F401  (asm: the module's fixture)


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


def test_cached_and_series_sweeps_load_everything_before_storing(asm):  # noqa: F811
    """The in-place steps that most boxes run (stores through the caches, the
    energy series): 27 population loads, then only stores. 45 of them in the
    line-aligned odd sweeps (test_isa_order), 27 otherwise; the series adds the
    five sums of a run, two of 16 bytes and one of 8."""
    cached = _kernels(asm, r"k_step_cachedILi\dELi\dELi[12]E")
    assert len(cached) == 3 * 8 * 2          # FP64, FP32, FP32-X; no FP16
    series = _kernels(asm, r"k_seriesILi\dELi\dELi[12]E")
    assert len(series) == 4 * 8 * 2
    for nm, ops in {**cached, **series}.items():
        aligned = re.search(r"ILi[03]ELi\dELi2E", nm) is not None
        sums = 3 if "k_series" in nm else 0
        assert all("load" in op for op in ops[:27]), nm
        assert all("store" in op for op in ops[27:]), nm
        assert len(ops) - 27 == (45 if aligned else 27) + sums, (nm, len(ops) - 27)
        if sums:
            assert sum(op.endswith("dwordx4") for op in ops[27:]) == 2, nm


def test_cached_series_and_pair_kernels_collide_with_the_step_s_arithmetic(asm):  # noqa: F811
    """Per storage form and variant, the floating-point instructions of the single
    step (test_isa_order holds the sweeps and the pool to one multiset) are those
    of the cached step; the series adds the same ones in every kernel of a
    storage form (velocity and energy sums), and the pair has them twice, but
    for integer divisions by way of FP32 and conversions of constants that its
    two collisions share."""
    def all_of(pattern):
        return re.findall(r"^(_ZN3kbc\S*" + pattern + r"\S*):", asm, flags=re.M)

    step = {re.search(r"k_stepILi(\d)ELi(\d)", nm).groups(): _fp_ops(asm, nm)
            for nm in all_of(r"k_stepILi\dELi\dELi0ELb0ELb0")}
    assert len(step) == 4 * 8
    names = all_of(r"k_step_cachedILi\dELi\dELi\dE")
    assert len(names) == 3 * 8 * 3
    for nm in names:
        ref = step[re.search(r"cachedILi(\d)ELi(\d)", nm).groups()]
        assert _fp_ops(asm, nm) == ref, nm
    names = all_of(r"k_seriesILi\dELi\dELi\dELb\d")
    assert len(names) == 4 * 8 * 3 + 8       # FP16 pull also on 64-node chunks
    extra = {}
    for nm in names:
        form, var = re.search(r"k_seriesILi(\d)ELi(\d)", nm).groups()
        ops, ref = _fp_ops(asm, nm), step[form, var]
        assert not ref - ops, nm
        assert ops - ref == extra.setdefault(form, ops - ref), nm
    names = all_of(r"k_pairILi\dELi\dELb\d")
    assert len(names) == 2 * 8 + 4           # FP64 past and through the caches, FP32 natural
    for nm in names:
        ref = step[re.search(r"k_pairILi(\d)ELi(\d)", nm).groups()]
        ops = _fp_ops(asm, nm)
        twice = Counter({op: 2 * n for op, n in ref.items()})
        more, less = ops - twice, twice - ops
        div = more.pop("v_cvt_f32_u32", 0)
        assert more.pop("v_mul_f32", 0) == div and more.pop("v_cvt_u32_f32", 0) == div and not more, (nm, more)
        assert set(less) <= {"v_cvt_f32_f64"}, (nm, less)
