"""The bucketed quadrature on rows whose ratios p / q lie far apart (cold drafts or targets, probabilities of any fp32
size), against direct pair sums or the exponential-sum rule in fp64.

Tolerance per entry: as for ordinary rows, r's fp32 rounding (6e-8), the parts' interpolation (7e-9) and the rounding of a
token's place in its part and of the polynomial's upper coefficients (5e-9): 8e-8.
Notation: p = target, q = draft.
"""
import pytest
import torch

import paper_2410_18234_amd as mdss
from test_gpu_bucket import law, rows, weights

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


def octaves(p, q):
    w = weights(p.double(), q.double())
    return float((w.amax(1) / w.masked_fill(w == 0, float("inf")).amin(1)).log2().max())


def cold_rows(B, V, seed, target, draft):
    """Softmax rows at the given temperatures of one set of logits (the draft's with noise, a second one warmer)."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    normal = lambda: torch.randn((B, V), generator=g, device=DEV, dtype=torch.float64)
    ell = 3.0 * normal()
    return [torch.softmax(x, 1).float() for x in (ell / target, (ell + normal()) / draft, (ell + normal()) / (1.5 * draft))]


# (octaves at least: past 32 the evaluation keeps a part of the row's polynomials in LDS, past 64 there are windows)
@pytest.mark.parametrize("B,V", [(3, 5001), (2, 33000), (1, 70003)])
@pytest.mark.parametrize("target,draft,least", [(1.0, 0.55, 32), (1.0, 0.45, 38), (1.0, 0.3, 66), (0.3, 1.0, 66), (0.4, 0.3, 40)])
def test_chunks_of_wide_rows(B, V, target, draft, least):
    p, q1, q2 = cold_rows(B, V, V + int(100 * draft), target, draft)
    assert octaves(p, q1) > least
    for K in (2, 3):
        check(mdss.induced_dist_expsum(p, q1, K), law(p, q1, None, K))
    check(mdss.induced_dist_pair_expsum(p, q1, q2), law(p, q1, q2, 2))


@pytest.mark.parametrize("B,V", [(3, 70001), (130, 9000)])
def test_one_wide_token(B, V):
    # a single probability below 2^-96 among ordinary ones; a chunk without any other weight; a chunk without any
    p, q, _ = rows(B, V, 600 + V)
    q[0, 5] = 1e-36
    p[1, V // 2] = 1e-40
    q[2, :4096] = 0.0
    q[2, 17] = 1e-38
    check(mdss.induced_dist_expsum(p, q, 2), law(p, q, None, 2))
    check(mdss.induced_dist_pair_expsum(p, q, q.flip(0)), law(p, q, q.flip(0), 2))


@pytest.mark.parametrize("V", [300000, 500001])
def test_many_chunks(V):
    # chunks of different octaves: a part of the row at weights 2^20 above the rest
    p, q, _ = rows(2, V, 700 + V)
    q[:, V // 2:] *= 2.0 ** -20
    check(mdss.induced_dist_expsum(p, q, 2), law(p, q, None, 2))


@pytest.mark.parametrize("B,V,times", [(8, 128256, 3.0), (8, 32000, 3.0), (256, 32000, 3.0), (256, 4000, 5.0)])
@pytest.mark.parametrize("draft", [0.5, 0.3])
def test_wide_rows_keep_their_form(B, V, times, draft):
    # Wide rows are summed and evaluated by all of a row's chunks, or from one workgroup's registers: at most three (rows
    # of a few us: five) times an ordinary row's time (1.3 to 2.5 measured; 4.8 to 10 in chunks and 3.2 in
    # registers when one workgroup streamed such a row).
    p, q, _ = cold_rows(B, V, 1, 1.0, draft)
    _, warm, _ = cold_rows(B, V, 1, 1.0, 1.0)
    r = torch.empty_like(p)
    ws = torch.empty(mdss.workspace_bytes_expsum(B, V, 2), dtype=torch.uint8, device=DEV)

    def median(q):
        taken = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                mdss.induced_dist_expsum(p, q, 2, r=r, workspace=ws)
            b.record()
            b.synchronize()
            taken.append(a.elapsed_time(b))
        return sorted(taken)[7]

    median(q)
    assert median(q) <= times * median(warm)


@pytest.mark.parametrize("B,V", [(3, 3001), (130, 9001), (128, 16385), (128, 32768)])
@pytest.mark.parametrize("target,draft", [(1.0, 0.3), (0.3, 1.0), (0.4, 0.3), (1.0, 0.17)])
def test_registers_of_wide_rows(B, V, target, draft):
    p, q1, q2 = cold_rows(B, V, V + int(100 * draft), target, draft)
    p[0, 3] = q1[1, 4] = q2[2, 5] = 0.0
    for K in (2, 4):
        check(mdss.induced_dist_expsum(p, q1, K), law(p, q1, None, K))
    if V < 10000:
        check(mdss.induced_dist_pair_expsum(p, q1, q2), law(p, q1, q2, 2))


def test_wide_rows_with_residual_sums():
    # the summed form's r is the plain call's and its sums are those of max(0, p - r), for both forms and bad rows
    for B, V in ((130, 9000), (3, 40001)):
        p, q, _ = cold_rows(B, V, V, 1.0, 0.3)
        q[1, 7] = float("nan")
        status = torch.full((B,), 99, dtype=torch.int32, device=DEV)
        acc = torch.empty(mdss.workspace_bytes_accept(B, V), dtype=torch.uint8, device=DEV)
        r = mdss.induced_dist_expsum_sums(p, q, 2, acc, row_status=status)
        assert torch.equal(r.nan_to_num(-1.0), mdss.induced_dist_expsum(p, q, 2).nan_to_num(-1.0))
        assert status.tolist() == [0, mdss.MDSS_ROW_BAD_PROB] + [0] * (B - 2)
        parts = (V + 1023) // 1024 * 4
        sums = acc.view(torch.float64)[:B * parts].view(B, parts)
        res = torch.zeros((B, parts * 256), dtype=torch.float64, device=DEV)
        res[:, :V] = (p.double() - r.double()).clamp(min=0.0)
        want = res.view(B, parts, 256).sum(2)
        assert bool(sums[1].isnan().all()) or bool(sums[1].sum().isnan())
        keep = torch.arange(B, device=DEV) != 1
        assert torch.allclose(sums[keep], want[keep], rtol=1e-12, atol=1e-300)


def test_longest_rows_stay_in_chunks():
    # a row past 6.3 M tokens would have more chunks than the merge takes: it must not be streamed by one workgroup instead
    taken = []
    for V in (3500000, 7000000):
        g = torch.Generator(device=DEV).manual_seed(V)
        p = torch.softmax(3.0 * torch.randn((1, V), generator=g, device=DEV), 1)
        q = torch.softmax(p.log() + torch.randn((1, V), generator=g, device=DEV), 1)
        r, ws = torch.empty_like(p), torch.empty(mdss.workspace_bytes_expsum(1, V, 2), dtype=torch.uint8, device=DEV)
        runs = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            mdss.induced_dist_expsum(p, q, 2, r=r, workspace=ws)
            b.record()
            b.synchronize()
            runs.append(a.elapsed_time(b))
        taken.append(sorted(runs)[3])
    assert taken[1] <= 4.0 * taken[0], taken


@pytest.mark.parametrize("B,V,s", [(1, 50257, 64), (3, 40000, 200), (8, 128256, 16)])
def test_three_drafts_of_a_small_support(B, V, s):
    p, q, _ = rows(B, V, 800 + V)
    top, at = torch.topk(q, s, dim=1)
    q = torch.zeros_like(q).scatter_(1, at, top / top.sum(1, keepdim=True))
    check(mdss.induced_dist(p, q, 3, s), law(p, q, None, 3))
    over = mdss.induced_dist(p, q, 3, s - 1)
    assert bool(over.isnan().all())


def test_host_threads_on_their_own_streams():
    # the launch sizes are looked up once per device by whichever thread comes first
    import threading

    cases = [cold_rows(3, 40000 + 128 * i, i, 1.0, 1.0)[:2] for i in range(4)]
    want = [mdss.induced_dist_expsum(p, q, 2) for p, q in cases]
    got, errors = [None] * len(cases), []
    start = threading.Barrier(len(cases))

    def work(i):
        try:
            p, q = cases[i]
            stream = torch.cuda.Stream(DEV)
            stream.wait_stream(torch.cuda.default_stream(DEV))
            with torch.cuda.stream(stream):
                r = torch.empty_like(p)
                ws = torch.empty(mdss.workspace_bytes_expsum(*p.shape, 2), dtype=torch.uint8, device=DEV)
                start.wait()
                for _ in range(20):
                    mdss.induced_dist_expsum(p, q, 2, r=r, workspace=ws)
            stream.synchronize()
            got[i] = r
        except Exception as e:  # seen by the main thread
            errors.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for r, w in zip(got, want):
        assert torch.equal(r, w)


@pytest.mark.parametrize("B,V", [(2, 100), (130, 6000), (2, 40000)])
@pytest.mark.parametrize("K", [2, 3, 6])
def test_widest_rows_within_the_range_rule(B, V, K):
    # 289 octaves, more than the registers' and the chunks' forms hold and within the 2^300 that is not flagged: the
    # streamed form, with and without the residual sums; 330 octaves are past the rule in every form
    g = torch.Generator(device=DEV).manual_seed(V)
    p = torch.softmax(3.0 * torch.randn((B, V), generator=g, device=DEV, dtype=torch.float64), 1)
    q = torch.softmax(p.log() + torch.randn((B, V), generator=g, device=DEV, dtype=torch.float64), 1)
    p[:, 3], q[:, 3] = 0.25, 2.0 ** -147
    p[:, V - 2], q[:, V - 2] = 2.0 ** -146, 0.125
    p[0, 5] = 0.0
    p, q = p.float(), q.float()
    assert 280 < octaves(p, q) < 300
    status = torch.zeros(B, dtype=torch.int32, device=DEV)
    r = mdss.induced_dist_expsum(p, q, K, row_status=status)
    assert int(status.abs().sum()) == 0
    check(r, law(p, q, None, K))
    acc = torch.empty(mdss.workspace_bytes_accept(B, V), dtype=torch.uint8, device=DEV)
    assert torch.equal(mdss.induced_dist_expsum_sums(p, q, K, acc, row_status=status), r)
    assert int(status.abs().sum()) == 0
    parts = (V + 1023) // 1024 * 4
    res = torch.zeros((B, parts * 256), dtype=torch.float64, device=DEV)
    res[:, :V] = (p.double() - r.double()).clamp(min=0.0)
    sums = acc.view(torch.float64)[:B * parts].view(B, parts)
    assert torch.allclose(sums, res.view(B, parts, 256).sum(2), rtol=1e-12, atol=1e-300)
    p[1, 3] = 2.0 ** 40
    r = mdss.induced_dist_expsum(p, q, K, row_status=status)
    assert status.tolist() == [0, mdss.MDSS_ROW_RANGE] + [0] * (B - 2)
    assert bool(r[1].isnan().all()) and not bool(r[0].isnan().any())
