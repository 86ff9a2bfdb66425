"""The bucketed quadrature on rows whose ratios p / q lie far apart (cold drafts or targets, probabilities of any fp32
size), against direct pair sums in fp64.

Tolerance per entry: as for ordinary rows, r's fp32 rounding (6e-8), the parts' interpolation (6e-9) and the rounding of a
token's place in its part and of the polynomial's upper coefficients (5e-9): 8e-8.
Notation: p = target, q = draft.
"""
import pytest
import torch

import paper_2410_18234_amd as mdss

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TOL = 8e-8


def pair_sums(p, q1, q2):
    """r in fp64 by the O(V^2) sums over drafted pairs (q2 None: two i.i.d. drafts from q1); no zero probabilities."""
    p, q1 = p.double(), q1.double()
    q2 = q1 if q2 is None else q2.double()
    w1, w2 = p / q1, p / q2
    out = [(q2[b] / (w1[b][:, None] + w2[b])).sum(1) + (q1[b] / (w2[b][:, None] + w1[b])).sum(1)
           for b in range(p.shape[0])]
    return p * torch.stack(out)


def check(r, ref, tol=TOL):
    assert bool(torch.isfinite(r).all())
    big = ref > 1e-30
    err = ((r.double() - ref).abs() / ref.clamp(min=1e-30))[big].max().item()
    assert err <= tol, err


def apart(B, V):
    """Ratios from 2^-138 to 2^220: a token of the smallest ratio, most of whose law comes from pairs with tokens of
    ratios 90 to 180 times its own."""
    q = torch.full((B, V), 0.5 / V)
    p = q * 2.0 ** -130 * torch.logspace(0, 1, V, base=2.0)
    p[:, 1], q[:, 1] = 2.0 ** -147, 2.0 ** -10.5
    p[:, 2], q[:, 2] = 2.0 ** 120, 2.0 ** -100
    return p.to(DEV), q.to(DEV)


@pytest.mark.parametrize("B,V", [(1, 64), (130, 64), (2, 5000)])
def test_ratios_hundreds_of_octaves_apart(B, V):
    p, q = apart(B, V)
    w = p.double() / q.double()
    assert float((w.max() / w.min()).log2()) > 340
    check(mdss.induced_dist(p, q, 2), pair_sums(p, q, None))
    check(mdss.induced_dist_pair(p, q, q.flip(0)), pair_sums(p, q, q.flip(0)))
