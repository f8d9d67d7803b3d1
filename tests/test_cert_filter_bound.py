"""The two bf16 filters in front of the certified FP32 scan never exclude a pair
whose canonical FP32 distance is at most the threshold.  numpy models of the
matrix-core sums (products of bf16 values, exact in fp32, added in several orders
with one fp32 rounding each, from the row's start value) are tested at the tightest
threshold, the pair's own canonical distance."""
import numpy as np
import pytest

F = np.float32


def bf16(x):
    """Round to bf16, nearest even (finite input)."""
    u = np.ascontiguousarray(x, F).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16 << 16).astype(np.uint32).view(F)


def canonical(q, x, metric):
    """fp32 sequential fma over ascending dimensions (float64 holds each fma's exact sum to 2^-53)."""
    r = np.zeros(q.shape[0], F)
    for j in range(q.shape[1]):
        if metric == 0:
            t = (q[:, j] - x[:, j]).astype(F).astype(np.float64)
            r = (t * t + r.astype(np.float64)).astype(F)
        else:
            r = (q[:, j].astype(np.float64) * x[:, j] + r.astype(np.float64)).astype(F)
    return r


def sum32(start, terms, order):
    acc = start.astype(F)
    cols = list(range(terms.shape[1]))
    if order == "reversed":
        cols = cols[::-1]
    if order == "pairwise":
        t = terms
        while t.shape[1] > 1:
            if t.shape[1] % 2:
                t = np.concatenate([t, np.zeros((t.shape[0], 1), F)], 1)
            t = (t[:, 0::2] + t[:, 1::2]).astype(F)
        return (acc + t[:, 0]).astype(F)
    for j in cols:
        acc = (acc + terms[:, j]).astype(F)
    return acc


def data(kind, rng, n, d):
    x = rng.standard_normal((n, d))
    if kind == "offset":
        x = 300 + x
    elif kind == "ints":
        x = rng.integers(0, 256, (n, d)).astype(np.float64)
    elif kind == "wide":
        x = x * 10.0 ** rng.uniform(-6, 6, (n, d))
    elif kind == "half_ulp":   # every value half way between two bf16 values, the worst rounding
        x = 2.0 ** rng.integers(-3, 4, (n, d)) * (1 + 2.0 ** -8)
    return x.astype(F)


@pytest.mark.parametrize("kind", ["normal", "offset", "ints", "wide", "half_ulp"])
@pytest.mark.parametrize("metric", [0, 1])
def test_filters_keep_every_pair_at_its_own_distance(kind, metric):
    worst = 0.0
    for d in (1, 2, 5, 32, 100, 256):
        rng = np.random.default_rng([31, d, metric, len(kind)])
        x = data(kind, rng, 400, d)
        q = np.where(rng.random((400, 1)) < 0.5, x * F(1 + 1e-3), data(kind, rng, 400, d)).astype(F)
        ca, cb = F(np.sqrt(F(d))) * F(2.0 ** -122), F(d) * F(2.0 ** -120)
        h0 = F(2) * (ca + cb)
        h1 = F(1.02 * 2.0 ** (-8 if metric == 0 else -9) + (12 * d + 64 if metric == 0 else 6 * d + 32) * 2.0 ** -24) + 2 * ca
        l1 = F((3.3 if metric == 0 else 1.7) * 2.0 ** -16 + (16 * d + 96 if metric == 0 else 8 * d + 48) * 2.0 ** -24) + 2 * ca
        ax = F(-0.5) * (F(1) - h1) if metric == 0 else h1
        xn, qn = np.zeros(400, F), np.zeros(400, F)
        for j in range(d):
            xn = (x[:, j].astype(np.float64) ** 2 + xn).astype(F)
            qn = (q[:, j].astype(np.float64) ** 2 + qn).astype(F)
        xh, qh = bf16(x), bf16(q)
        xl, ql = bf16((x - xh).astype(F)), bf16((q - qh).astype(F))
        r = canonical(q, x, metric)
        thd = r if metric == 0 else -r
        bq = F(0.5) * ((F(1) - h1) * qn - h0 - thd) if metric == 0 else -thd - h0 - h1 * qn
        first = np.concatenate([xh * qh, xh * ql], 1)
        for order in ("ascending", "reversed", "pairwise"):
            acc = sum32((ax * xn).astype(F), first, order)
            assert not (acc < bq).any(), (kind, metric, d, order)
            acc = sum32(acc, xl * qh, order)
            dot = (acc - ax * xn).astype(F)
            v = (qn + xn - 2 * dot).astype(F) if metric == 0 else -dot
            e = (l1 * (qn + xn) + h0).astype(F)
            assert not ((v - e).astype(F) > thd).any(), (kind, metric, d, order)
            worst = max(worst, float(np.max(np.abs(v - thd) / np.maximum(e, F(1e-30)))))
    assert worst < 1.0
    if kind == "half_ulp":   # the bound is not idle: half of it would exclude pairs that belong
        acc = sum32((F(-0.5) * xn if metric == 0 else np.zeros_like(xn)), first, "ascending")
        tight = 0.25 * 2.0 ** (-8 if metric == 0 else -9) * (xn + qn)
        full = F(0.5) * (qn - thd) if metric == 0 else -thd
        assert (acc < full - tight).any() or (acc > full + tight).any()
