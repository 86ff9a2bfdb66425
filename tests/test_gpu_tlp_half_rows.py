"""The half tail's plan where its selection can go wrong: rows shorter than s and than a workgroup, unaligned rows, equal
keys, and rows whose first-ranked tokens all lie with a few threads (more candidates than the list holds).
Notation: p = target, q1 / q2 = draft distributions."""
import numpy as np
import pytest

from oracle import tlp
from test_gpu_tlp import check_plan, gpu_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [2, 5, 63, 1021, 4096, 32768, 50257, 600000])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("s", [1, 8])
def test_half_rows(V, two, s):
    rng = np.random.default_rng(V + two)
    B = 5
    z = 3.0 * rng.standard_normal((B, V))
    p = np.exp(z)
    q1 = np.exp(z + rng.standard_normal((B, V)))
    q2 = np.exp(0.5 * (z + rng.standard_normal((B, V))))
    p[1], q1[1], q2[1] = 1.0, 1.0, 1.0                  # every key equal
    p[2] = rng.integers(1, 4, V)                        # many equal keys
    few = np.arange(V) % 4096 < 32                      # the tokens of eight threads
    p[3] = np.where(few, 10.0 + rng.random(V), rng.random(V))
    p, q1, q2 = ((x / x.sum(1, keepdims=True)).astype(np.float32) for x in (p, q1, q2))
    g = gpu_plan(p, q1, q2 if two else None, s, tlp.HALF)
    check_plan(p, q1, q2 if two else None, s, tlp.HALF, g)
