"""The sorted tail's plan where its cells can go wrong: rows of one and of several groups, unaligned rows, equal keys
(within a cell, and more than a cell holds), keys of both signs, keys in few bins.
Notation: p = target, q1 / q2 = draft distributions."""
import numpy as np
import pytest

from oracle import tlp
from test_gpu_tlp import check_plan, gpu_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [2, 63, 4097, 12288, 16385, 32000, 50257, 131073])
@pytest.mark.parametrize("two", [False, True])
def test_cells(V, two):
    rng = np.random.default_rng(V + two)
    B = 8
    z = 3.0 * rng.standard_normal((B, V))
    p = np.exp(z)
    q1 = np.exp(z + rng.standard_normal((B, V)))
    q2 = np.exp(0.5 * (z + rng.standard_normal((B, V))))
    p[1], q1[1], q2[1] = 1.0, 1.0, 1.0                            # every key equal
    p[2] = rng.integers(1, 9, V)                                  # many equal keys
    p[3] = 1.0 + 1e-6 * rng.random(V)                             # one bin
    p[4, rng.random(V) < 0.01] = 0.0                              # negative keys
    p[5, V // 2:], q1[5, V // 2:], q2[5, V // 2:] = 0.0, 0.0, 0.0  # half the row at key 0
    p[6] = np.floor(p[6] * 4) + 1.0                               # some equal keys
    p, q1, q2 = ((x / x.sum(1, keepdims=True)).astype(np.float32) for x in (p, q1, q2))
    g = gpu_plan(p, q1, q2 if two else None, 5, tlp.SORTED)
    check_plan(p, q1, q2 if two else None, 5, tlp.SORTED, g)
