"""The built objects keep no state between calls but what is documented: with several devices or threads in a process,
anything remembered from one call may be wrong for the next (reads the symbol tables of this repository's own builds)."""
import re
import subprocess

import pytest

from paper_2403_12422_amd import build

ALLOWED = {
    # the scratch of jf_layernorm_q_bwd_static and its address per device, the test hook for tile shapes, the error code of
    # each thread; a constant table of functions
    build.LIB: ("scratch", "g_scratch_ptr", "g_scratch_mutex", "g_forced_shape", "g_last_hip_error", "launch_gemm.*table"),
    # the exception class and the module's own tables
    build.EXT: ("g_error", "g_methods", "g_module"),
}


@pytest.mark.parametrize("path", ALLOWED)
def test_no_state_between_calls(path):
    nm = subprocess.run(["nm", "--defined-only", path], capture_output=True, text=True, check=True, timeout=60).stdout
    rows = [line.split()[1:3] for line in nm.splitlines()]
    # this repository's variables (kernel handles are named like functions of the namespace, with parameters)
    own = [m for kind, m in rows if kind in "bBdD" and re.match(r"_ZL|_ZG?V?Z*N?2jfL?|_ZG?V?Z*N?12_GLOBAL__N_1", m) and "kernelEP" not in m]
    assert own
    unknown = [m for m in own if not re.search("|".join(ALLOWED[path]), m)]
    assert not unknown, unknown
