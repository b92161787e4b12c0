"""The backward of a residual connection -- LayerNorm backward, Add, Dropout -- against the oracle's: every difference has to start at a
rounding tie.  A code that falls to the other side of a tie is one code off; where the next operator finds it among the largest
values of a block, that block's scale moves by up to one part in a hundred, and with it codes of the block that are at no tie."""
import numpy as np

import oracle
from parity import REL_TOL, assert_codes_close, assert_scales_close, expand

P = 0.1


def inputs(g, N, C, block):
    """Quantized operands; the gradient that Add takes is largest where dX lies nearest to a tie, one place in each block, so that a
    code which differs there is the largest of its sum."""
    from paper_2403_12422_amd import workloads
    x, gamma, _, gr = workloads.layernorm_case(int(g.integers(1 << 30)), N, C)
    (X, SX), (G, SG) = oracle.quantize_block(x, block), oracle.quantize_block(gr, block)
    mean, rstd = oracle.layernorm_q(X, SX, gamma, np.zeros(C, np.float32), 1e-5, block)[2:4]
    q, s, _, _, dx = oracle.layernorm_q_bwd(G, SG, X, SX, gamma, mean, rstd, block)
    ratio = np.abs(dx) / expand(s.astype(np.float64), block)
    near = np.abs(ratio - np.floor(ratio) - 0.5) + (ratio < 1)
    blocks = near.reshape(N // block, block, C // block, block).transpose(0, 2, 1, 3).reshape(-1, block * block)
    R = np.zeros_like(blocks, np.int8)
    R[np.arange(len(R)), blocks.argmin(1)] = 127
    R = R.reshape(N // block, C // block, block, block).transpose(0, 2, 1, 3).reshape(N, C)
    R = np.ascontiguousarray(R * np.sign(dx).astype(np.int8))
    bits, _ = workloads.dropout_mask_bits(g, N, C, P)
    return dict(G=(G, SG), X=(X, SX), gamma=gamma, mean=mean, rstd=rstd, R=(R, s), bits=bits)


def chain(i, block, layernorm=None, add=None, dropout=None):
    """[(codes, scales, values before rounding)] of the three operators; by the oracle where no other is given."""
    a = (layernorm or _layernorm)(i, block)
    b = (add or (lambda *t: oracle.add_q(*t, block)))(*a[:2], *i["R"])
    c = (dropout or (lambda q, s: oracle.dropout_q(q, s, i["bits"], P, block)))(*b[:2])
    return [(t[0], t[1], t[-1]) for t in (a, b, c)]


def _layernorm(i, block):
    return oracle.layernorm_q_bwd(*i["G"], *i["X"], i["gamma"], i["mean"], i["rstd"], block)


def check(got, want, block, inputs_of):
    """Both chains with the same operands; inputs_of(k, codes, scales): the oracle's operator k on these results of the one before.
    Returns the number of blocks whose scale a tie has moved."""
    blocks = lambda m: m.reshape(m.shape[0] // block, block, m.shape[1] // block, block).any((1, 3))
    moved, before = 0, np.zeros_like(want[0][1], bool)   # blocks in which the operator before has a code on the other side
    for k, ((q, s), (oq, os_, o64)) in enumerate(zip([t[:2] for t in got], want)):
        name = ("LayerNorm backward", "Add", "Dropout")[k]
        rel = np.abs(s.astype(np.float64) - os_) / np.maximum(os_, 1e-300)
        far = rel > REL_TOL
        assert not (far & ~before).any(), f"{name}: the scale of a block moved with no code of its input on the other side of a tie"
        moved += int(far.sum())
        clean = expand(~before, block)
        assert_codes_close(np.where(clean, q, oq), oq, name, prequant=o64, scales=os_, block=block)
        if k:   # the rest, and all of it: the operator is right about what it was given
            tq, ts, t64 = inputs_of(k, *got[k - 1][:2])
            assert_scales_close(s, ts, name)
            assert_codes_close(q, tq, name, prequant=t64, scales=ts, block=block)
        before = before | blocks(q != oq)
    return moved


def oracle_operator(i, block):
    def run(k, q, s):
        o = oracle.add_q(q, s, *i["R"], block) if k == 1 else oracle.dropout_q(q, s, i["bits"], P, block)
        return o[0], o[1], o[-1]
    return run
