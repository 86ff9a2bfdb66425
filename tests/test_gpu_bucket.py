"""The bucketed quadrature (csrc/bucket.hip) at the sizes where its form changes: rows held in one
workgroup's registers (up to 4096, 16384 and 32768 tokens), rows split into chunks, rows streamed
window by window, aligned and unaligned, against the same law in fp64 (plain torch, an
exponential-sum rule at half the step on a grid cut at 1e-17).

Tolerance per entry: r's fp32 rounding (6e-8), the parts' interpolation (7e-9) and the rounding of
p / q's place in its part and of the polynomial's upper coefficients (5e-9): 8e-8.
Notation: p = target, q = draft.
"""
import math

import pytest
import torch

import paper_2410_18234_amd as mdss

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
TOL = 8e-8


def rows(B, V, seed, sigma=3.0, noise=1.0, temp=1.0, zeros=0.0):
    g = torch.Generator(device=DEV).manual_seed(seed)

    def normal():
        return torch.randn((B, V), generator=g, device=DEV, dtype=torch.float64)

    ell = sigma * normal()
    p, q1, q2 = torch.softmax(ell, 1), torch.softmax((ell + noise * normal()) / temp, 1), torch.softmax(
        (ell + noise * normal()) / (1.5 * temp), 1)
    if zeros:
        p = p * (torch.rand((B, V), generator=g, device=DEV) >= zeros)
        q1 = q1 * (torch.rand((B, V), generator=g, device=DEV) >= zeros)
        p[:, 0] = 0.5
        q1[:, 0] = 0.25
    return p.float(), q1.float(), q2.float()


def weights(p, q):
    return torch.where(q > 0, p / torch.where(q > 0, q, torch.ones_like(q)), torch.zeros_like(p))


def law(p, q1, q2, K):
    """r in fp64 (q2 None: K i.i.d. drafts from q1)."""
    p, q1 = p.double(), q1.double()
    q2 = q1 if q2 is None else q2.double()
    w1, w2, acc, h = weights(p, q1), weights(p, q2), torch.zeros_like(p), 0.25
    pos = torch.cat((w1[w1 > 0], w2[w2 > 0]))
    t0, t1 = math.log(1e-17 / (K * float(pos.max()))), math.log(45.0 / float(pos.min()))
    two = q2 is not q1
    for k in range(math.floor(t0 / h), math.ceil(t1 / h) + 1):
        a = math.exp(k * h)
        e1, e2 = torch.exp(-a * w1), torch.exp(-a * w2)
        S1, S2 = (q1 * e1).sum(1, keepdim=True), (q2 * e2).sum(1, keepdim=True)
        acc += h * a * (e1 * (q1 > 0) * S2 + e2 * (q2 > 0) * S1) if two else K * h * a * e1 * S1 ** (K - 1)
    zero = p == 0
    z1, z2 = (q1 * zero).sum(1, keepdim=True), (q2 * zero).sum(1, keepdim=True)
    if two:
        return torch.where(zero, 0.5 * (q1 * z2 + q2 * z1), p * acc)
    return torch.where(q1 > 0, torch.where(zero, q1 * z1 ** (K - 1), p * acc), torch.zeros_like(p))


def check(r, ref, tol):
    assert bool(torch.isfinite(r).all())
    big = ref > 1e-30
    err = ((r.double() - ref).abs() / ref.clamp(min=1e-30))[big].max().item()
    assert err <= tol, err
    assert bool((r[~big] <= 1e-29).all())


@pytest.mark.parametrize("B,V,K", [(3, 2, 2), (130, 4096, 3), (2, 4097, 8), (130, 4099, 2), (129, 16384, 2),
                                   (128, 16387, 4), (128, 32768, 2), (2, 32768, 2), (1, 32769, 5), (130, 33001, 2),
                                   (1, 70003, 2)])
def test_one_law(B, V, K):
    p, q, _ = rows(B, V, 100 + V)
    check(mdss.induced_dist_expsum(p, q, K), law(p, q, None, K), TOL)
    if K == 2:
        # the same kernels; the chunks of a long row follow each call's own workspace size
        check(mdss.induced_dist(p, q, 2), law(p, q, None, 2), TOL)


@pytest.mark.parametrize("B,V", [(2, 3), (130, 4096), (2, 4097), (128, 16384), (128, 16388), (3, 40001)])
def test_two_laws(B, V):
    p, q1, q2 = rows(B, V, 200 + V)
    check(mdss.induced_dist_pair_expsum(p, q1, q2), law(p, q1, q2, 2), TOL)


@pytest.mark.parametrize("B,V,K", [(2, 5000, 2), (130, 5000, 3), (3, 40000, 2)])
def test_zero_probabilities(B, V, K):
    p, q1, q2 = rows(B, V, 300 + V, zeros=0.3)
    check(mdss.induced_dist_expsum(p, q1, K), law(p, q1, None, K), TOL)
    check(mdss.induced_dist_pair_expsum(p, q1, q2), law(p, q1, q2, 2), TOL)


@pytest.mark.parametrize("B,V,temp", [(3, 3001, 0.25), (130, 20000, 0.2), (2, 40001, 0.3)])
def test_weights_past_one_window(B, V, temp):
    # a cold draft: weights spanning more than the 64 octaves held in LDS, drafts below 2^-96
    p, q1, q2 = rows(B, V, 400 + V, temp=temp)
    w = weights(p.double(), q1.double())
    assert float((w.amax(1) / w.masked_fill(w == 0, math.inf).amin(1)).log2().max()) > 66
    check(mdss.induced_dist_expsum(p, q1, 2), law(p, q1, None, 2), TOL)
    check(mdss.induced_dist_pair_expsum(p, q1, q2), law(p, q1, q2, 2), TOL)


@pytest.mark.parametrize("V", [16, 5000, 40000])
def test_equal_laws(V):
    # p = q: one bucket holds the row, r = q (K = 2: every pair splits evenly)
    p, _, _ = rows(3, V, 500 + V)
    s = p.double().sum(1, keepdim=True)
    check(mdss.induced_dist_expsum(p, p, 2), p.double() * s, TOL)


def test_offsets_into_a_buffer():
    # rows at an odd 4-byte offset take the unaligned loads: the same bits as the aligned ones
    p, q, _ = rows(4, 6000, 7)
    pad = torch.zeros(4 * 6000 + 1, device=DEV)
    pu, qu = pad.clone()[1:].view(4, 6000), pad.clone()[1:].view(4, 6000)
    pu.copy_(p)
    qu.copy_(q)
    assert torch.equal(mdss.induced_dist_expsum(p, q, 2), mdss.induced_dist_expsum(pu, qu, 2))
