"""The minimum-distortion decode's tie rule on the GPU (paper Sec. 3.2; the
paper leaves ties open, the reading taken is: among equal path metrics the
predecessor with the smallest state index, then the smallest final state).

Inputs are dyadic (codewords in {-3..3}/4, weights in {-6..6}/8), so every
fp64 distortion and every metric sum is exact on both sides and exact ties
are everywhere: the states must equal the oracle's bit for bit (the
oracle's rule is pinned against path enumeration on tiny shapes), and
w_hard must be codebook[states].
"""
import sys

import numpy as np
import pytest

import paper_2605_10655_amd as P
from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P.load_library()
    yield


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def host(t):
    return t.detach().cpu().numpy()


def dyadic(seed, B, L, S, V=1):
    r = np.random.default_rng(seed)
    c = (r.integers(-3, 4, (S, V) if V > 1 else S) / 4.0).astype(np.float32)
    w = (r.integers(-6, 7, (B, L)) / 8.0).astype(np.float32)
    return w, c


@pytest.mark.parametrize("n,k,B,L", [
    (2, 1, 9, 14), (6, 1, 7, 12), (10, 1, 5, 11), (14, 1, 3, 9),
    (4, 2, 9, 13), (8, 2, 7, 12), (12, 2, 5, 10), (13, 2, 3, 9), (16, 2, 3, 9),
    (6, 3, 6, 10), (9, 3, 4, 8), (14, 3, 2, 7),
])
def test_scalar_viterbi_tie_rule(n, k, B, L):
    w, c = dyadic(17 * n + k, B, L, 1 << n)
    _say(f"[ties] scalar n={n} k={k} B={B} L={L}")
    st, wh = P.viterbi_decode(dev(w), dev(c), n, k)
    torch.cuda.synchronize()
    st, wh = host(st), host(wh)
    rst, cost = O.viterbi(w, c, n, k)
    np.testing.assert_array_equal(st, rst)
    np.testing.assert_array_equal(wh, c[st])
    # the inputs really tie: some step has several states of the best metric
    m = O.maxmarginal_gap(w, c, n, k, rst)
    assert np.any(m == 0.0)


@pytest.mark.parametrize("n,B,L", [(8, 6, 12), (12, 4, 10), (16, 2, 8)])
def test_vector_viterbi_tie_rule(n, B, L):
    w, c = dyadic(31 * n, B, L, 1 << n, V=2)
    _say(f"[ties] vector n={n} V=2 B={B} L={L}")
    st, wh = P.bcjr_vec_viterbi_decode(dev(w), dev(c), n, 4, 2)
    torch.cuda.synchronize()
    st, wh = host(st), host(wh)
    rst, _ = O.viterbi(w, c, n, 4, V=2)
    np.testing.assert_array_equal(st, rst)
    np.testing.assert_array_equal(wh, c[st].reshape(B, L))
    assert np.any(O.maxmarginal_gap(w, c, n, 4, rst, V=2) == 0.0)


def _strict_less_decode(w, c, n, k):
    """Plain fp64 recursion: among the predecessors in order the first value,
    then any strictly smaller one; a NaN that comes first stays."""
    S, K = 1 << n, 1 << k
    G = S >> k
    cd = c.astype(np.float64)
    out = np.zeros(w.shape, np.int64)
    for b in range(w.shape[0]):
        M = np.zeros(G)
        digits = []
        for t in range(w.shape[1]):
            F = (float(w[b, t]) - cd) ** 2 + np.repeat(M, K)
            if t == w.shape[1] - 1:
                fin = np.where(F < np.inf, F, np.inf)
                s = int(np.argmin(fin)) if np.isfinite(fin).any() else 0
            else:
                F = F.reshape(K, G)
                M, d = F[0].copy(), np.zeros(G, np.int64)
                for j in range(1, K):
                    less = F[j] < M
                    M, d = np.where(less, F[j], M), np.where(less, j, d)
                digits.append(d)
        for t in range(w.shape[1] - 1, -1, -1):
            out[b, t] = s
            if t:
                v = s >> k
                s = int((digits[t - 1][v] << (n - k)) | v)
    return out


@pytest.mark.parametrize("n,k", [(8, 2), (13, 2), (14, 1), (16, 2), (14, 3)])
@pytest.mark.parametrize("bad", [None, "nan", "inf"])
def test_scalar_viterbi_nonfinite_codewords(n, k, bad):
    # equality is exact: the recursion is one square and one sum in fp64 on
    # both sides (dyadic values, no rounding)
    B, L = 2, 257 if (n, k) in ((14, 1), (16, 2)) else 7  # (the longer rows take the form with the minimum too)
    w, c = dyadic(5 * n + k, B, L, 1 << n)
    w[1, 2] = np.inf
    if bad:
        r = np.random.default_rng(n)
        c[r.integers(0, 1 << n, 1 << (n - 3))] = np.nan if bad == "nan" else np.inf
    _say(f"[ties] non-finite codewords n={n} k={k} {bad}")
    with np.errstate(invalid="ignore"):
        want = _strict_less_decode(w, c, n, k)
    st, _ = P.viterbi_decode(dev(w), dev(c), n, k)
    assert np.array_equal(host(st), want)
