"""The register checks of test_pinned_registers.py for the kernels with records of
long terms, which a second compilation of the same sources holds: their Jacobian
rows live in registers that the compiler must not touch, like the others."""
import os
import subprocess

import pytest

import tests.test_pinned_registers as base
from paper_1505_00383_amd import build as B


def _compile(tmp_path_factory, src):
    kept = B.kept_asm(src, long=True)
    if kept:
        with open(kept) as f:
            return f.read()
    if not os.path.exists(base.HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / (src + ".s")
    cmd = [base.HIPCC, "-x", "hip"] + B.COMMON + B.DEVICE + B.LONG_FLAGS + [
        "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def test_pinned_row(tmp_path_factory):
    asm = _compile(tmp_path_factory, "eval.hip")
    base.test_pinned_registers_untouched_by_compiler(asm, r"_ZN2ph25eval_d_pinned_long_kernel\S*", 128, "256")


@pytest.mark.parametrize("src,kernel", [("eval_dd.hip", "_ZN2ph24eval_dd_arow_long_kernel"),
                                        ("eval_qd.hip", "_ZN2ph24eval_qd_arow_long_kernel")])
def test_accumulation_register_row(tmp_path_factory, src, kernel):
    base.test_accumulation_register_row_untouched_by_compiler((_compile(tmp_path_factory, src), kernel))


@pytest.mark.parametrize("src", B.LONG_UNITS)
def test_build_compiles_the_checked_unit(src):
    """What is checked is what is linked: the build has one object of each unit,
    compiled with the flags that the check uses."""
    assert [(o, e) for s, o, e in B.sources() if s == src] == [(src + ".o", []), (os.path.join("long", src + ".o"),
                                                                                 B.LONG_FLAGS)]
