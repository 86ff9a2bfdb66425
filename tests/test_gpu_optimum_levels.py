"""The optimal acceptance where its levels can go wrong: rows at and past the register-held length, unaligned rows, rows
that leave few, many or too many candidates (ranked whole), ratios at the ends of the fp32 range, masses outside the
fixed-point range.  Notation: p = target, q = draft."""
import numpy as np
import pytest

from test_gpu_optimum import check, gpu_opt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [2, 255, 4097, 32768, 32769, 70000])
@pytest.mark.parametrize("K", [2, 5])
def test_levels(V, K):
    rng = np.random.default_rng(V + K)
    B = 12
    z = 3.0 * rng.standard_normal((B, V))
    p = np.exp(z)
    q = np.exp(z + rng.standard_normal((B, V)))
    p[1] = q[1] = 1.0                                   # one ratio
    p[2] = q[2] * (1.0 + 1e-3 * rng.random(V))          # all tokens in one bin
    p[3] = q[3] * np.exp(60.0 * rng.random(V) - 30.0)   # ratios over 86 octaves
    q[4, rng.random(V) < 0.5] = 0.0
    p[5, rng.random(V) < 0.5] = 0.0
    q[6, V // 2:] = 0.0
    q[6, 0] = 1.0
    p[5, 0] = q[4, 0] = 1.0
    p /= p.sum(1, keepdims=True)
    q /= q.sum(1, keepdims=True)
    p[7] *= 4.0                                         # masses outside [2^-6, 2]: ranked whole
    q[8] *= 1e-5
    q[9, V // 2:] *= 1e-34                              # ratios past the fp32 range, subnormal drafts
    p, q = p.astype(np.float32), q.astype(np.float32)
    ps, ks, st = gpu_opt(p, q, K)
    check(p, q, K, ps, ks, st)
