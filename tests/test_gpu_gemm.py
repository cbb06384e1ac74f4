"""The fp32 contractions against 64 bits.

On a graph of self-loops only a one-layer GCN is its contraction: logits = X W + b, and the weight
gradient is X^T dY with the dY that the pass leaves.  Every matrix step adds to a sum with an error of
at most 2^-23 of it (the matrix cores round down), six steps for 16 k; the split itself leaves out
2^-25 of a product.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (rows, d_in, d_out): edges of the 64- and 128-wide tiles and of the steps of 16 k, widths of no whole
# vector, 64-wide tiles up to 1280 of them and 128-wide ones beyond, one short of and over a split
CASES = [
    (1, 1, 1), (1, 4, 4), (63, 16, 64), (64, 17, 65), (65, 15, 47), (127, 32, 128), (129, 33, 129), (128, 8, 130),
    (200, 31, 3), (300, 61, 77), (1000, 100, 256), (40960, 20, 128), (40961, 20, 128), (81921, 36, 64), (90000, 64, 172),
    (50021, 136, 40), (2049, 300, 200),
]


def run(n, din, dout, edit=None):
    from paper_2605_11517_amd import Session
    print("case gemm %d %d %d" % (n, din, dout), flush=True)
    rng = np.random.default_rng([n, din, dout])
    X = rng.standard_normal((n, din)).astype(np.float32)
    W = rng.standard_normal((din, dout)).astype(np.float32)
    b = rng.standard_normal(dout).astype(np.float32)
    if edit:
        edit(X, W)
    y = rng.integers(0, dout, n).astype(np.int32)
    m = np.ones(n, dtype=np.uint8)
    s = Session("gcn", [din, dout], np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), 1, "random", 1, X,
                [dict(W=W, b=b)], y, m)
    s.epoch()
    return X, W, b, s.results()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d" % c)
def test_contractions_against_64_bits(case):
    n, din, dout = case
    X, W, b, r = run(n, din, dout)
    X64, W64 = X.astype(np.float64), W.astype(np.float64)

    def check(got, ref, absolute, k):
        steps = 6 * -(-k // 16) + 2
        assert np.all(np.abs(got - ref) <= steps * 2.0 ** -23 * absolute)
        # (rounding errors of both signs: far below the bound; measured 1.1e-7 to 2.6e-7)
        assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(absolute) / np.sqrt(max(1, min(k, 4)))
        return steps

    check(r["act"][-1], X64 @ W64 + b, np.abs(X64) @ np.abs(W64) + np.abs(b), din)
    dY = np.asarray(r["gact"][-1], dtype=np.float64)
    check(r["gW"][0], X64.T @ dY, np.abs(X64).T @ np.abs(dY), n)


def test_infinities_nan_and_overflow_are_those_of_fp32():
    def edit(X, W):
        X[3, 2] = np.inf
        X[70, 0] = np.nan
        X[90, 39] = -np.inf
        X[100] = 0
        X[100, 1] = np.float32(3.4028e38)      # rounds up to infinity in bfloat16
        W[1] = np.float32(0.5)
        W[5, 7] = np.inf

    X, W, b, r = run(150, 40, 70, edit)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = (X.astype(np.float64) @ W.astype(np.float64) + b).astype(np.float32)
    got = r["act"][-1]
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref)
    assert np.allclose(got[ok], ref[ok], rtol=1e-5, atol=1e-4)
