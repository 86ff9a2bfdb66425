"""The truncated alphabet at the edges of its kernels: rows at and past the register-held length, unaligned rows, bins
and ties of more entries than are ranked in LDS, and draws from units of several tiles.  Notation: p = target."""
import numpy as np
import pytest
import torch

import paper_2410_18234_amd as mdss
from oracle import alphabet
from test_gpu_alphabet import check_truncate, gpu_truncate
from test_gpu_parity import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [2, 257, 4099, 32768, 32769, 70000])
@pytest.mark.parametrize("m", [1, 300, 2500])
def test_truncate_edges(V, m):
    rng = np.random.default_rng(V + m)
    p = rng.dirichlet(np.full(V, 0.3), size=5).astype(np.float32)
    p[1] = np.float32(1.0 / V)                                  # every entry tied, cut by id
    p[2] = np.float32(2.0 ** -8) * (1 + np.arange(V) % 3000 * np.float32(2.0 ** -23))  # one bin, low bits differ
    p[3, rng.random(V) < 0.5] = np.float32(3.0 / V)             # a tie block across the row
    p[4, m // 2:] = 0.0                                         # fewer positive entries than m
    pt, mass, st = gpu_truncate(p, m)
    check_truncate(p, m, pt, mass, st)


@pytest.mark.parametrize("V", [3, 256, 4097, 40004, 262144, 262145, 600000])
def test_post_units(V):
    rng = np.random.default_rng(V)
    B, m = 16, min(20, V - 1)
    p = (rng.random((B, V)) + 0.1).astype(np.float32)
    p[:, rng.random(V) < 0.3] = 0.0
    p[:, -1] = 1.0
    p /= p.sum(1, keepdims=True)
    pt, mass, _ = alphabet.truncate(p, m)
    u2 = np.stack([np.full(B, 0.9999999), rng.integers(0, 1 << 24, B) / float(1 << 24)], 1).astype(np.float32)
    u2[0, 1], u2[1, 1] = 0.0, 1.0 - 2.0 ** -24
    z = np.zeros(B, np.int32)
    out, kept = mdss.alphabet_post(dev(p), dev(pt), dev(mass), dev(z), dev(u2))
    out, kept = out.cpu().numpy(), kept.cpu().numpy()
    oout, okept = alphabet.post(p, pt > 0, mass, z, u2)
    np.testing.assert_array_equal(kept, okept)
    for b in np.flatnonzero(kept == 0):
        assert pt[b, out[b]] == 0 and p[b, out[b]] > 0
        # the token's own interval of the complement's distribution holds the uniform, but for fp64 sums' rounding
        comp = np.where(pt[b] > 0, 0.0, p[b].astype(np.float64))
        C, t = np.cumsum(comp), float(u2[b, 1]) * comp.sum()
        assert C[out[b]] - comp[out[b]] <= t * (1 + 1e-12) and C[out[b]] >= t * (1 - 1e-12)
