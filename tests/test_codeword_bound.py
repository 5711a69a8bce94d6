"""The error bound behind the codes decided on the matrix units, checked on the CPU with numpy's fp16 and fp32.

A point's block x and a codeword c, both scaled by the power of two that takes the quantiser's largest codeword component below 1, are
split into a high and a low fp16 half each; <x, c> - |c|^2 / 2 is formed as xl ch + xh cl + xh ch, the norm in two halves, in fp32.  The
largest of four codewords in a row keeps its value but for the 5 low bits, which take its number, and which of the four it is
is decided by the same products with 2 bits for the number.  Every such value is to lie within 2^-17 (|x|^2 + C) of (|x|^2 - d) / 2, d the distance
that encode's chain of fused multiply-adds forms and C the largest |c|^2, so that a lead of 2^-16 (|x|^2 + C) is a true one
(csrc/pq.hpp: pq_encode_kernel).
"""
import numpy as np
import pytest

F, H = np.float32, np.float16


def _values(X, C, low=True):
    """(values in fp32, (|x|^2 - d) / 2 in fp64, the bound, d), scaled: X [n][ds], C [256][ds]."""
    scale = F(2.0) ** F(-np.frexp(np.abs(C).max())[1])
    x, c = (X * scale).astype(F), (C * scale).astype(F)
    xh, ch = x.astype(H).astype(F), c.astype(H).astype(F)
    xl, cl = (x - xh).astype(H).astype(F), (c - ch).astype(H).astype(F)
    if not low:
        xl, cl = 0 * xl, 0 * cl
    c2, x2 = np.zeros(len(C), F), np.zeros(len(X), F)
    for t in range(X.shape[1]):
        c2 = (c2.astype(np.float64) + c[:, t].astype(np.float64) ** 2).astype(F)
        x2 = (x2.astype(np.float64) + x[:, t].astype(np.float64) ** 2).astype(F)
    nh = F(-0.5) * c2
    acc = np.broadcast_to(nh.astype(H).astype(F) + (nh - nh.astype(H).astype(F)).astype(H).astype(F), (len(X), len(C))).astype(F)
    d = np.zeros((len(X), len(C)), F)
    for t in range(X.shape[1]):
        for a, b in ((xl, ch), (xh, cl), (xh, ch)):
            acc = acc + a[:, t, None] * b[None, :, t]             # (products of halves are exact in fp32)
        u = (x[:, t, None] - c[None, :, t]).astype(F)
        d = (d + u.astype(np.float64) ** 2).astype(F)
    exact = ((x.astype(np.float64) ** 2).sum(1)[:, None] - d) / 2
    return acc, exact, 2.0 ** -17 * (x2 + c2.max()).astype(np.float64), d


def _numbered(v, bits, number):
    return ((v.view(np.uint32) & ~np.uint32((1 << bits) - 1)) | number.astype(np.uint32)).view(F)


def _decide(X, C, band_factor=2.0, **kw):
    """(sure, code) as the kernel has them, (lowest, second-lowest are left to the chain), and the chain's code."""
    acc, exact, bound, d = _values(X, C, **kw)
    band = band_factor * bound
    # fours of a lane half: codewords 8 j .. 8 j + 3 and 8 j + 4 .. 8 j + 7
    fours = acc.reshape(len(X), 64, 4).max(2)
    fours = _numbered(fours, 5, np.broadcast_to(np.arange(64) // 2, fours.shape))
    order = np.sort(fours, 1)
    at = fours.argmax(1)
    inside = np.take_along_axis(acc.reshape(len(X), 64, 4), at[:, None, None], 1)[:, 0]
    inside = _numbered(np.ascontiguousarray(inside), 2, np.broadcast_to(np.arange(4), inside.shape))
    two = np.sort(inside, 1)
    sure = (order[:, -1].astype(np.float64) - order[:, -2] > band) & (two[:, -1].astype(np.float64) - two[:, -2] > band)
    return sure, 4 * at + inside.argmax(1), d.argmin(1), (acc, exact, bound, fours, inside, at)


def _blocks(kind, ds, rng, n=1500):
    C = rng.standard_normal((256, ds))
    X = C[rng.integers(0, 256, n)] + 0.5 * rng.standard_normal((n, ds))
    if kind == "scales":                                       # codewords and points of very different size
        C, X = C * np.exp2(rng.integers(-20, 1, (256, 1))), X * np.exp2(rng.integers(-12, 12, (n, 1)))
    if kind == "between":                                      # points halfway between two codewords
        X = (C[rng.integers(0, 256, n)] + C[rng.integers(0, 256, n)]) / 2
    if kind == "close":                                        # codewords that differ in their last bits
        C = C[:1] + 2.0 ** -13 * C
        X = C[rng.integers(0, 256, n)]
    if kind == "large":                                        # points as large as the halves hold
        X = 2.0 ** 14 * X
    return X.astype(F), C.astype(F)


@pytest.mark.parametrize("ds", [4, 6, 8, 12, 16])
@pytest.mark.parametrize("kind", ["gauss", "scales", "between", "close", "large"])
def test_values_stay_within_the_bound_and_sure_codes_are_the_chains(kind, ds):
    X, C = _blocks(kind, ds, np.random.default_rng(ds))
    sure, code, chain, (acc, exact, bound, fours, inside, at) = _decide(X, C)
    rows = np.arange(len(X))
    assert (np.abs(acc - exact) <= bound[:, None]).all()
    best = exact.reshape(len(X), 64, 4)
    assert (np.abs(fours - best.max(2)) <= bound[:, None]).all()
    assert (np.abs(inside - best[rows, at]) <= bound[:, None]).all()
    assert (code[sure] == chain[sure]).all()
    if kind == "gauss":
        assert sure.mean() > 0.99


def test_the_lead_is_needed():
    """Without it the number in the low bits, and without the low halves their loss, decide wrongly."""
    wrong = lambda X, C, **kw: (lambda t: int((t[0] & (t[1] != t[2])).sum()))(_decide(X, C, **kw))
    X, C = _blocks("close", 6, np.random.default_rng(1))
    assert wrong(X, C) == 0 and wrong(X, C, band_factor=0.0) > 0
    X, C = _blocks("between", 8, np.random.default_rng(2))
    acc, exact, bound, _ = _values(X, C, low=False)
    assert not (np.abs(acc - exact) <= bound[:, None]).all()
