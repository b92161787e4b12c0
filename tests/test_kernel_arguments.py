"""Structures through which kernels read their argument segment belong to the kernels' parameter lists: with a parameter more in front of
what is read, in the kernel and at its launch, the sources do not compile (host code; nothing is run)."""
import glob
import os
import shutil
import subprocess

import pytest

from paper_2403_12422_amd.build import CSRC, INCLUDE

# file, the end of a parameter list and what is passed for it, the source that launches the kernel
KERNELS = {
    "gemm_kernel": ("jf_gemm_kernel.hpp", ("const v4i sizes, const GemmResults)", "const v4i sizes, int, const GemmResults)"),
                    ("tiles}, results_of(a))", "tiles}, 0, results_of(a))"), "jf_gemm_fwd_b32.hip"),
    "gemm_pair_kernel": ("jf_gemm_kernel.hpp", ("const int8_t* X, const v2u64, const float*, const GemmResults", "const int8_t* X, const v2u64, const float*, const float*, const GemmResults"),
                         ("a2.SB, results_of(a1)", "a2.SB, a2.SB, results_of(a1)"), "jf_gemm_bwd_pair_b32.hip"),
    "gemm_wide_pair_kernel": ("jf_gemm_wide.hpp", ("gemm_wide_pair_kernel(const GemmArgs, const GemmArgs", "gemm_wide_pair_kernel(const GemmArgs, const int, const GemmArgs"),
                              ("st, a1, a2, t1", "st, a1, 0, a2, t1"), "jf_gemm_bwd_pair_b64.hip"),
    "layernorm_rows_kernel": ("jf_layernorm_rows.hpp", ("int layout, int wgs, const LayerNormRows)", "int layout, int wgs, const float*, const LayerNormRows)"),
                              ("waves), grid, a)", "waves), grid, a.beta, a)"), "jf_layernorm_rows_b32.hip"),
    "layernorm_bwd_rows_kernel": ("jf_layernorm_rows.hpp", ("const float* gamma, const LayerNormBwdRows)", "const float* gamma, const float*, const LayerNormBwdRows)"),
                                  ("a.row_wgs, a.gamma, a)", "a.row_wgs, a.gamma, a.mean, a)"), "jf_layernorm_rows_b32.hip"),
}


def _compiles(csrc, source):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-fsyntax-only", "-w", "-I", str(csrc), "-I", INCLUDE,
                          str(csrc / source)], capture_output=True, text=True, timeout=120)
    return res.returncode == 0, res.stdout + res.stderr


@pytest.mark.parametrize("kernel", KERNELS)
def test_a_parameter_more_does_not_compile(kernel, tmp_path):
    name, parameters, passed, source = KERNELS[kernel]
    for f in glob.glob(os.path.join(CSRC, "*.h*")):
        shutil.copy(f, tmp_path)
    ok, out = _compiles(tmp_path, source)
    assert ok, out
    text = (tmp_path / name).read_text()
    for old, new in (parameters, passed):
        assert text.count(old) == 1, old
        text = text.replace(old, new)
    (tmp_path / name).write_text(text)
    ok, out = _compiles(tmp_path, source)
    assert not ok and "static assertion failed" in out.replace("static_assert failed", "static assertion failed"), out
