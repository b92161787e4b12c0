"""LayerNorm backward -> Add -> Dropout, each on what the one before has left, against the oracle's chain (run with -m gpu): one pass over
whole rows at every block size, the kernels for wider rows, and the two-kernel scheme."""
import numpy as np
import pytest

import layernorm_chain as lc
import paper_2403_12422_amd as jf
from paper_2403_12422_amd import workloads
from test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,N,C", [(32, 2080, 1280), (32, 16384, 480), (32, 5120, 2304), (32, 256, 2304), (64, 10240, 704), (64, 512, 1344),
                                       (128, 20480, 384)])
def test_differences_start_at_ties(block, N, C):
    say(f"chain block={block} {N} x {C}")
    i = lc.inputs(workloads.rng(9900 + C), N, C, block)
    call = lambda f: lambda *t: [*map(host, f(*map(dev, t)))] + [None]
    got = lc.chain(i, block, layernorm=lambda i, b: call(lambda *t: jf.jf_layernorm_q_bwd(*t, b))(*i["G"], *i["X"], i["gamma"], i["mean"], i["rstd"]),
                   add=call(lambda *t: jf.jf_add_q(*t, block)), dropout=call(lambda q, s: jf.jf_dropout_q(q, s, dev(i["bits"]), lc.P, block)))
    want = lc.chain(i, block)
    moved = lc.check(got, want, block, lc.oracle_operator(i, block))
    say(f"  {int(np.count_nonzero(got[0][0] != want[0][0]))} codes of dX on the other side of a tie, {moved} scales behind it moved")
