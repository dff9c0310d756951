"""The mathematics behind estimating rows without a full sort (CPU check, numpy only).

The GPU kernel puts a row, scaled to integers q counted from its minimum, into value buckets of 2^sh, and
knows for every bucket the number of smaller elements, their sum and the sum of its own offsets.  D is
T^2/n plus n times G(i) = (P - i T/n)^2 / (i (n - i)), which does not change when every value is shifted.
With j of a bucket's c elements below the split, P is at least L(j) = max(S_b + j lo, S_e - (c - j) hi) for the
bucket's limits lo and hi, and P - i T/n is at most 0, so G is at most its value on those two lines; it is convex
along each, so its maximum there is at the bucket's start, its end or where the lines cross.  The kernel
evaluates the three points in fp32 and keeps the buckets whose bound reaches the best bucket end less a margin of
4e-6 of D.  This test follows that evaluation in numpy float32, step by step, and compares it with the exact G at
every position: the errors of a bound and of the best end together have to stay inside the margin.
"""
import numpy as np
import pytest

F = np.float32
MARGIN = F(4e-6)
# threads, buckets and the longest row of the kernels' classes
CLASSES = [(256, 512, 768), (256, 1024, 1792), (256, 512, 2304), (512, 2048, 4608), (256, 1024, 4608), (256, 2048, 9216),
           (512, 2048, 13312), (256, 2048, 13312)]
KINDS = ["gauss", "mixture", "laplace", "one_sided", "student_t", "two_maxima", "far_mean", "outlier", "uniform", "few_values"]


def draw(rng, kind, n):
    g = rng.standard_normal(n)
    w = {"gauss": lambda: 0.05 * g + 0.01,
         "mixture": lambda: np.where(rng.random(n) < 0.7, 0.3, -0.7) * 0.04 + 0.02 * g,
         "laplace": lambda: rng.laplace(0.004, 0.03, n),
         "one_sided": lambda: np.abs(g) + 0.25,
         "student_t": lambda: rng.standard_t(3, n),
         "two_maxima": lambda: np.concatenate([h := rng.standard_t(2.2, n // 2), -h, np.zeros(n % 2)]),
         "far_mean": lambda: 1e-3 * g + 3.0,
         "outlier": lambda: np.where(np.arange(n) == n // 3, 40.0, g),
         "uniform": lambda: rng.uniform(-1, 1, n),
         "few_values": lambda: np.round(g * 8) / 8}[kind]()
    return w.astype(F)


def fma(a, b, c):
    return F(a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64))


def buckets(w, NB):
    """Scaled integers, sorted; their shift; the bucket of each."""
    ex = int(np.frexp(np.abs(w).max())[1])
    q = np.rint(np.ldexp(w.astype(np.float64), 48 - ex)).astype(np.int64)
    low = q.min()
    off = 2 - low + (low & 1)
    q = np.sort(q + off)
    sh = max(35, int(q[-1] >> 32).bit_length() + 32 - (NB.bit_length() - 1))
    assert q[0] >= 2 and q[-1] >> sh < NB
    return q, off, sh, (q >> sh).astype(np.int64)


def kernel_bounds(q, sh, b, NB, threads):
    """ub and the value at the end of every bucket, as the kernel forms them; bucket counts."""
    n, per = len(q), NB // threads
    c = np.bincount(b, minlength=NB)
    offs = np.zeros(NB, np.int64)
    np.add.at(offs, b, q - (b << sh))
    sums = np.zeros(NB, np.int64)
    np.add.at(sums, b, q)
    below_n, below_s = np.cumsum(c) - c, np.cumsum(sums) - sums
    mean, nf = float(q.sum()) / n, F(n)
    bf = F(F(offs >> 24) * F(2.0 ** (24 - sh)))
    first = np.arange(threads) * per

    def spread(Q, i):
        return F(F(Q * Q) * F(F(1) / np.maximum(F(i * F(nf - i)), F(0.5))))
    Q0 = F(np.ldexp(below_s[first].astype(np.float64) - below_n[first] * mean, -sh))
    i0 = F(below_n[first])
    g0, dist = spread(Q0, i0), F(first - np.ldexp(mean, -sh))
    ub, end = np.empty(NB, F), np.empty(NB, F)
    for k in range(per):
        at = first + k
        ck = F(c[at])
        js, i1 = F(ck - bf[at]), F(below_n[at] + c[at])
        Q1 = F(Q0 + fma(ck, dist, bf[at]))
        g1, gs = spread(Q1, i1), spread(fma(js, dist, Q0), F(i0 + js))
        ub[at], end[at] = np.maximum(np.maximum(g0, g1), gs), g1
        Q0, i0, g0, dist = Q1, i1, g1, F(dist + F(1))
    return ub, end, c, mean


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("threads,NB,n", CLASSES)
def test_bound_holds_within_the_margin_and_prunes(kind, threads, NB, n):
    rng = np.random.default_rng(100 * n + KINDS.index(kind))
    for n in (n, n - 37):
        q, off, sh, b = buckets(draw(rng, kind, n), NB)
        ub, end, c, mean = kernel_bounds(q, sh, b, NB, threads)
        # exact G in units of a bucket's width, at positions 1 .. n-1 (whole sums fit the long double's 64 bits)
        P = np.cumsum(q)[:-1].astype(np.longdouble)
        i = np.arange(1, n).astype(np.longdouble)
        G = np.ldexp(P - i * (np.longdouble(q.sum()) / n), -sh) ** 2 / (i * (n - i))
        inside = np.full(NB, -np.inf)                     # over a bucket's positions, its end among them
        np.maximum.at(inside, b[:-1], G.astype(np.float64))
        used = np.flatnonzero(c)
        ends = used[np.cumsum(c)[used] <= n - 1]
        gbest = end[ends].max()
        mean_f = F(np.ldexp(mean - float(off), -sh))
        margin = F(MARGIN * F(gbest + F(mean_f * mean_f)))
        short = (inside[used] - ub[used].astype(np.float64)).max()            # a bound below what it bounds
        over = float(gbest) - inside.max()                                    # an end value above the maximum
        assert max(short, 0.0) + max(over, 0.0) <= 0.5 * float(margin), (short, over, margin)
        alive = ub >= F(gbest - margin)
        assert alive[b[:-1][G == G.max()]].all()
        if kind in ("gauss", "mixture", "laplace", "one_sided", "uniform"):
            assert c[alive & (c > 0)].sum() <= max(320, n // 20)              # (a list or two; 100 in a bucket at a Laplacian's peak)


def test_joint_convexity_of_the_score():
    """D(i, P) is convex along arbitrary segments of the (i, P) plane (0 < i < n)."""
    rng = np.random.default_rng(3)
    n, T = 1000.0, 37.5
    for _ in range(2000):
        i1, i2 = rng.uniform(1, n - 1, 2)
        P1, P2 = rng.uniform(-200, 200, 2)
        t = rng.uniform(0, 1)
        D = lambda P, i: P * P / i + (T - P) ** 2 / (n - i)
        mid = D(t * P1 + (1 - t) * P2, t * i1 + (1 - t) * i2)
        assert mid <= t * D(P1, i1) + (1 - t) * D(P2, i2) + 1e-9 * (abs(mid) + 1)
