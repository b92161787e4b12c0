"""The check of the residual connection's backward itself, on chains of the oracle in which a mistake is planted."""
import numpy as np
import pytest

import layernorm_chain as lc
import oracle
from paper_2403_12422_amd import workloads
from parity import expand

B = 32


def _case():
    g = workloads.rng(9900)
    i = lc.inputs(g, 128, 160, B)
    return i, lc.chain(i, B)


def _flipped(i, nearest):
    """LayerNorm backward with one code moved over the tie nearest to its value: the nearest tie of all blocks, or one far away."""
    q, s, _, _, dx = lc._layernorm(i, B)
    ratio = np.abs(dx) / expand(s.astype(np.float64), B)
    off = np.abs(ratio - np.floor(ratio) - 0.5) + (ratio < 2) + (ratio > 120)
    at = np.unravel_index((off if nearest else -off * (off < 1)).argmin(), off.shape)
    away = np.floor(ratio[at]) + np.ceil(ratio[at]) - np.abs(q[at].astype(int))
    q = q.copy()
    q[at] = np.sign(q[at]) * int(away)
    return q, s, None, None, dx


def test_a_tie_may_move_a_scale():
    i, want = _case()
    got = lc.chain(i, B, layernorm=lambda i, b: _flipped(i, True))
    assert np.count_nonzero(got[0][0] != want[0][0]) == 1
    assert lc.check(got, want, B, lc.oracle_operator(i, B)) >= 1


def test_same_chain():
    i, want = _case()
    assert lc.check(lc.chain(i, B), want, B, lc.oracle_operator(i, B)) == 0


@pytest.mark.parametrize("mistake", ["code", "scale", "add code", "dropout scale"])
def test_mistakes_are_found(mistake):
    i, want = _case()
    with_code = lambda t: (np.where(np.arange(t[0].size).reshape(t[0].shape) == 5, t[0] + (1 - 2 * (t[0] > 0)), t[0]).astype(np.int8), *t[1:])
    with_scale = lambda t: (t[0], t[1] * np.float32(1.001), *t[2:])
    ops = {"code": dict(layernorm=lambda i, b: _flipped(i, False)), "scale": dict(layernorm=lambda i, b: with_scale(lc._layernorm(i, b))),
           "add code": dict(add=lambda *t: with_code(oracle.add_q(*t, B))),
           "dropout scale": dict(dropout=lambda q, s: with_scale(oracle.dropout_q(q, s, i["bits"], lc.P, B)))}[mistake]
    with pytest.raises(AssertionError):
        lc.check(lc.chain(i, B, **ops), want, B, lc.oracle_operator(i, B))
