"""GPU parity of the linear-domain kernels below 65536 states
(lin_group_kernel, lin_sg_kernel): every (state bits, k) shape they serve, at
block lengths around their chunks of steps (one lane chunk is 2 to 64 steps, a
batch of moments 2 or 4), with block counts that leave a wave's last blocks
empty, and blocks they mark for the log-domain repair pass (weights outside
the codebook's range) among ordinary ones.  Everything is compared with the
fp64 oracle.

Tolerances as everywhere: w_soft |err| <= 2e-5, logZ 1e-4 relative (of 1 where
logZ is smaller: it crosses zero at short blocks), gradients 1e-4 of
max(|ref_i|, rms(ref)) over the call's whole output; where the blocks are built
to leave the number range, with the bound that the repair pass's fp32 sets.
"""
import sys

import numpy as np
import pytest

import paper_2605_10655_amd as P
from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(n, 1) for n in range(2, 15)] + [(n, 2) for n in range(4, 16)] + [(n, 3) for n in range(6, 15)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P.load_library()
    yield


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def grad_err(gpu, ref):
    ref = np.asarray(ref, np.float64)
    rms = np.sqrt(np.mean(ref * ref))
    scale = np.maximum(np.abs(ref), rms)
    return float((np.abs(gpu.astype(np.float64) - ref) / np.where(scale > 0, scale, 1.0)).max())


def check(w, c, g, n, k, T, dc, tag, rows=slice(None)):
    ws, lz, dW, dC = P.bcjr_soft_codeword_fwd_vjp(dev(w), dev(c), n, k, T, dev(g), want_dCodebook=dc)
    soft, lz0 = P.bcjr_soft_codeword(dev(w), dev(c), n, k, T)
    ows, olz, odW, odC = O.soft_codeword_vjp(w, c, n, k, T, g)
    ws, soft, lz, lz0, dW = (x.cpu().numpy()[rows] for x in (ws, soft, lz, lz0, dW))
    ows, olz, odW = ows[rows], olz[rows], odW[rows]
    den = np.maximum(np.abs(olz), 1.0)
    e = [float(np.abs(ws - ows).max()), float(np.abs(soft - ows).max()), float((np.abs(lz - olz) / den).max()),
         float((np.abs(lz0 - olz) / den).max()), grad_err(dW, odW)]
    if dc:
        e.append(grad_err(dC.cpu().numpy(), odC))
    print(f"[lin-small] {tag} errors {['%.1e' % x for x in e]}", file=sys.__stderr__, flush=True)
    assert e[0] <= 2e-5 and e[1] <= 2e-5
    assert max(e[2:5]) <= 1e-4
    assert not dc or e[5] <= 1e-4


@pytest.mark.parametrize("n,k", SHAPES)
def test_shapes_and_lengths_match_oracle(n, k):
    r = np.random.default_rng(100 * n + k)
    c = r.standard_normal(1 << n).astype(np.float32)
    for L, B, T, dc in ((1, 3, 0.1, True), (2, 5, 0.3, True), (7, 37, 0.05, False),
                        (66, 3, 0.1, True), (129, 5 if n < 12 else 2, 0.05, True), (130, 3, 0.25, False)):
        # (at k = 1 the linear-domain kernels serve from T = 0.06 to 0.1 on, by form)
        w = r.standard_normal((B, L)).astype(np.float32)
        g = r.standard_normal((B, L)).astype(np.float32)
        check(w, c, g, n, k, T, dc, f"n={n} k={k} L={L} B={B} T={T} dc={dc}")


@pytest.mark.parametrize("n,k", [(4, 2), (7, 1), (8, 2), (9, 3), (10, 2), (12, 2), (13, 3), (14, 2), (15, 2)])
@pytest.mark.parametrize("dc", [False, True])
def test_far_and_marked_blocks(n, k, dc):
    """Blocks 1 and 4 hold weights far outside the codebook, whose distance the
    exponents leave out; every weight of block 2 lies beyond that (over 4096
    log2 units), which marks it: neither the others' results nor the sum over
    blocks may see what the first pass made of it.  (At 40 the log-domain
    pass itself resolves w_soft to 1e-4 only, so block 2 is not compared;
    with g = 0 its part of dCodebook is 0.)"""
    r = np.random.default_rng(7 * n + k)
    c = r.standard_normal(1 << n).astype(np.float32)
    w = r.standard_normal((6, 40)).astype(np.float32)
    w[1, 5] = -14.0
    w[4, 20] = 15.0
    w[2, :] = 40.0
    w[5, [3, 17]] = [6.0, -6.0]
    g = r.standard_normal((6, 40)).astype(np.float32)
    g[2, :] = 0.0
    check(w, c, g, n, k, 0.1, dc, f"far n={n} k={k} dc={dc}", rows=[0, 1, 3, 4, 5])


def test_non_finite_weights_stay_in_their_block():
    """A NaN weight marks its block alone: the other blocks of the wave keep
    the results they have without it."""
    r = np.random.default_rng(3)
    n, k = 6, 2
    c = r.standard_normal(1 << n).astype(np.float32)
    w = r.standard_normal((9, 33)).astype(np.float32)
    g = r.standard_normal((9, 33)).astype(np.float32)
    a = P.bcjr_soft_codeword_fwd_vjp(dev(w), dev(c), n, k, 0.1, dev(g), want_dCodebook=False)
    w[4, 10] = np.nan
    b = P.bcjr_soft_codeword_fwd_vjp(dev(w), dev(c), n, k, 0.1, dev(g), want_dCodebook=False)
    keep = [0, 1, 2, 3, 5, 6, 7, 8]
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x[keep], y[keep])
    assert not torch.isfinite(b[0][4]).all()


def call(w, c, g, n, k, T, dc, nbytes=None):
    """The fused call in a workspace filled with 0xFF; with its outputs the
    flags of the blocks, which the linear-domain kernels leave behind the
    scaled codebook: 1 for a block they marked (another value there: another
    kernel family ran)."""
    B, L = w.shape
    if nbytes is None:
        nbytes = P.bcjr_workspace_bytes(B, L, n, k, P.OP_FWD_VJP)
    work = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda:0")
    out = P.bcjr_soft_codeword_fwd_vjp(dev(w), dev(c), n, k, T, dev(g), want_dCodebook=dc, workspace=work)
    torch.cuda.synchronize()
    at = (4 * len(c) + 255) // 256 * 256
    return [None if x is None else x.cpu().numpy() for x in out], work[at:at + 4 * B].view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("n,k", [(2, 1), (4, 2), (8, 2), (8, 1), (9, 3), (10, 3), (11, 2), (12, 2), (15, 2)])
@pytest.mark.parametrize("T", [0.25, 1.0])
def test_any_gradient_scale(n, k, T):
    """The gradients are linear in g and a power of two is taken out of every
    block's g exactly: each block's g times its own 2^x yields the same bits
    of dW times 2^x, and the whole g times 2^x those of dCodebook (entries in
    the subnormal range carry one rounding there).  No block is marked, so
    all of it is the linear-domain kernels' own."""
    r = np.random.default_rng(13 * n + k)
    c = r.standard_normal(1 << n).astype(np.float32)
    B, L = 320 if n < 8 else 12, 70
    w = r.standard_normal((B, L)).astype(np.float32)
    g = r.standard_normal((B, L)).astype(np.float32)

    def run(gr, dc):
        out, flags = call(w, c, gr, n, k, T, dc)
        assert not flags.any()
        return out[2:]

    print(f"[lin-small] gradient scales n={n} k={k} T={T}", file=sys.__stderr__, flush=True)
    dW = run(g, False)[0]
    x = r.choice([-90, -50, -20, 0, 16, 24, 36, 60, 100], (B, 1))
    got = run(np.ldexp(g, x), False)[0]
    assert (np.abs(got - np.ldexp(dW, x)) <= 2.0 ** (np.maximum(x, 0) - 149)).all()
    dW, dC = run(g, True)
    for e in (-60, -30, 20, 36, 100):
        a, b = run(np.ldexp(g, e), True)
        tol = 2.0 ** (max(e, 0) - 149)
        assert (np.abs(a - np.ldexp(dW, e)) <= tol).all() and (np.abs(b - np.ldexp(dC, e)) <= tol).all()


@pytest.mark.parametrize("n,k", SHAPES)
def test_small_batches_run_the_same_kernels(n, k):
    """Batches that leave a wave's last blocks empty, down to one block, run the
    linear-domain kernels as large ones do: their flags say so, and every
    output has the bits that it has inside a batch of 130."""
    r = np.random.default_rng(17 * n + k)
    c = r.standard_normal(1 << n).astype(np.float32)
    w = r.standard_normal((130, 21)).astype(np.float32)
    g = r.standard_normal((130, 21)).astype(np.float32)
    at = (4 << n) + 255 & -256

    def soft(x):
        work = torch.full((P.bcjr_workspace_bytes(len(x), 21, n, k, P.OP_FWD),), 255, dtype=torch.uint8, device="cuda:0")
        out = P.bcjr_soft_codeword(dev(x), dev(c), n, k, 0.25, workspace=work)
        return [y.cpu().numpy() for y in out], work[at:at + 4 * len(x)].view(torch.int32).cpu().numpy()

    runs = [soft] + [lambda x, dc=dc: call(x, c, g[:len(x)], n, k, 0.25, dc) for dc in (False, True)]
    for i, run in enumerate(runs):
        big, marks = run(w)
        assert set(marks) <= {0, 1}, "the batch of 130"
        for B in (1, 3, 31):
            out, flags = run(w[:B])
            assert np.array_equal(flags, marks[:B]), f"call {i}, B = {B}"
            for a, b in zip(out[:3], big[:3]):
                np.testing.assert_array_equal(a, b[:B])


def lost_path(n, k, seed):
    """Blocks of 12 weights at T = 0.25 (2.885 log2 units per unit of squared
    distance) on a codebook that tells only whether a state's last two digits
    are 0.  Weight 0 lies on the codewords of (x, 0) and over 126 units from
    all others of its kind, weights 1 and 2 on those of (x, y) and 83 units from
    (0, 0): the best path begins with a step of 137 units, whose exponential is
    0 in fp32, the best without it has two steps of 83."""
    r = np.random.default_rng(seed)
    s = np.arange(1 << n)
    p, q = (s >> k) % (1 << k) > 0, s % (1 << k) > 0
    c = np.select([~p & ~q, ~p & q, p & ~q], [0.0, 8.9, 2.0], -5.364)
    w = np.zeros((5, 12))
    w[[1, 3], 0], w[[1, 3], 1:3] = 2.0, -5.364
    w[3, 8], w[3, 9:11] = 2.0, -5.364      # and the same inside the block
    c, w = c + 0.01 * r.standard_normal(1 << n), w + 0.01 * r.standard_normal(w.shape)
    return w.astype(np.float32), c.astype(np.float32), r.standard_normal(w.shape).astype(np.float32)


@pytest.mark.parametrize("n,k", SHAPES)
def test_a_path_that_both_sweeps_lose_marks_its_block(n, k):
    """Both sweeps lose the best path alike and their masses agree on the
    second best: only the size of alpha H shows it.  (The codewords of a kind
    are nearly alike, so that the gradients are small: their bound is the tangents'
    rounding, 2^-22 |g D| of a weight at distance D, times D / T.)"""
    w, c, g = lost_path(n, k, 23 * n + k)
    ref = O.soft_codeword_vjp(w, c, n, k, 0.25, g)
    assert ref[0][1, 0] > 8.0  # (the second best starts at 2)
    tol = 2.0 ** -22 * np.abs(g).max() * 9.0 ** 2 / 0.25
    soft = P.bcjr_soft_codeword(dev(w), dev(c), n, k, 0.25)
    assert np.abs(soft[0].cpu().numpy() - ref[0]).max() <= 2e-5
    for dc in (False, True):
        out, flags = call(w, c, g, n, k, 0.25, dc)
        assert flags.tolist() == [0, 1, 0, 1, 0]
        assert np.abs(out[0] - ref[0]).max() <= 2e-5
        assert np.abs(out[1] - ref[1]).max() <= 1e-4 * np.abs(ref[1]).max()
        for a, b in zip(out[2:], ref[2:]):
            assert a is None or np.abs(a - b).max() <= tol + 1e-4 * np.abs(b).max()


@pytest.mark.parametrize("n,k,T,served", [
    (5, 1, 0.064, ""), (5, 1, 0.066, "soft dw dc"), (9, 1, 0.074, ""), (9, 1, 0.076, "dc"), (10, 1, 0.059, ""),
    (10, 1, 0.084, "dc"), (8, 1, 0.086, "soft dw dc"),
    (6, 2, 0.039, ""), (6, 2, 0.041, "soft dw dc"), (12, 2, 0.022, ""), (12, 2, 0.023, "soft"),
    (11, 3, 0.039, ""), (12, 3, 0.023, "soft")])
def test_temperatures_that_the_linear_kernels_serve(n, k, T, served):
    """On each side of the lines of the dispatch (where ordinary weights begin to
    leave the kernels' number range), each form against the oracle."""
    r = np.random.default_rng(n + k)
    c = r.standard_normal(1 << n).astype(np.float32)
    w = r.standard_normal((3, 20)).astype(np.float32)
    g = r.standard_normal((3, 20)).astype(np.float32)
    ref = O.soft_codeword_vjp(w, c, n, k, float(np.float32(T)), g)
    at = (4 << n) + 255 & -256
    for form in ("soft", "dw", "dc"):
        if form == "soft":
            work = torch.full((P.bcjr_workspace_bytes(3, 20, n, k, P.OP_FWD),), 255, dtype=torch.uint8, device="cuda:0")
            out = [x.cpu().numpy() for x in P.bcjr_soft_codeword(dev(w), dev(c), n, k, T, workspace=work)]
            flags = work[at:at + 12].view(torch.int32).cpu().numpy()
        else:
            out, flags = call(w, c, g, n, k, T, form == "dc")
        assert (set(flags) <= {0, 1}) == (form in served.split()), form
        assert np.abs(out[0] - ref[0]).max() <= 2e-5
        for a, b in zip(out[2:], ref[2:]):
            assert a is None or grad_err(a, b) <= 1e-4


def clusters(n, k, B, L, marked):
    """Codewords about +-7.5 and weights on them; in the blocks `marked` the
    weights lie about 0, inside the codebook's range but 160 log2 units (at
    T = 0.25) from every codeword, below the floor of the vectors."""
    r = np.random.default_rng(31 * n + k)
    c = r.standard_normal(1 << n) + 7.5 * r.choice([-1.0, 1.0], 1 << n)
    c[:2] = -7.5, 7.5
    w = r.standard_normal((B, L)) + 7.5 * r.choice([-1.0, 1.0], (B, L))
    w[marked] = 0.3 * r.standard_normal((len(marked), L))
    return w.astype(np.float32), c.astype(np.float32), r.standard_normal((B, L)).astype(np.float32)


def repair_bounds(w, c, marked, T):
    """What the fp32 log-domain pass resolves of marked blocks: its local fields,
    k2 (w - c)^2 log2 units, round twice by 2^-24 of themselves, which changes
    probabilities by that times ln 2, and w_soft by that times the distance
    between the clusters; a missing or doubled repair is of the order of 1."""
    k2 = 1.4426950408889634 / (2 * T)
    d = np.abs(w[marked]).max() + np.median(np.abs(c))
    rel = 2.0 ** -23 * np.log(2.0) * k2 * d * d
    return rel, rel * 2 * np.median(np.abs(c))


@pytest.mark.parametrize("n,k", [(2, 1), (5, 1), (8, 1), (12, 1), (4, 2), (6, 2), (8, 2), (9, 2), (10, 2), (12, 2),
                                 (14, 2), (15, 2), (6, 3), (9, 3), (10, 3), (13, 3)])
def test_marked_blocks_are_recomputed(n, k):
    """Marked blocks among others (of the same wave and workgroup too): every
    output of the repair pass, and dCodebook as the sum of both passes', against
    the oracle; and in ever smaller workspaces, whose slots both passes use
    again, the same bits (dCodebook is summed in another order in fp64) until
    the log-domain kernels take over."""
    T, marked, B = 0.25, [0, 3, 4, 8], 9
    w, c, g = clusters(n, k, B, 20, marked)
    ref = O.soft_codeword_vjp(w, c, n, k, T, g)
    rest = [b for b in range(B) if b not in marked]
    rel, tol = repair_bounds(w, c, marked, T)
    full = P.bcjr_workspace_bytes(B, 20, n, k, P.OP_FWD_VJP)
    for dc in (False, True):
        out, flags = call(w, c, g, n, k, T, dc)
        assert flags[marked].all() and set(flags) <= {0, 1} and not flags.all()
        assert np.abs(out[0][rest] - ref[0][rest]).max() <= 2e-5
        assert np.abs(out[0] - ref[0]).max() <= 2e-5 + tol
        assert np.abs(out[1] / ref[1] - 1).max() <= 1e-4
        # (means over pairs of probabilities: twice the relative change, and
        # dCodebook's over the distance of up to 2 x 7.5 / T beside g)
        assert grad_err(out[2], ref[2]) <= 1e-4 + 2 * rel
        if dc:
            assert grad_err(out[3], ref[3]) <= 1e-4 + 30 * rel
        ran = 0
        for part in (0.75, 0.5, 0.35, 0.25, 0.15):
            try:
                less, fl = call(w, c, g, n, k, T, dc, int(full * part))
            except P.BcjrError as e:
                assert e.status == -3
                continue
            if not set(fl) <= {0, 1}:
                continue
            ran += 1
            assert np.array_equal(fl, flags)
            for a, b in zip(less[:3], out[:3]):
                np.testing.assert_array_equal(a, b)
            if dc:
                np.testing.assert_allclose(less[3], out[3], rtol=2.0 ** -22, atol=2.0 ** -22 * np.abs(out[3]).max())
        print(f"[lin-small] repair n={n} k={k} dc={dc}: {ran} smaller workspaces", file=sys.__stderr__, flush=True)
    soft = P.bcjr_soft_codeword(dev(w), dev(c), n, k, T)
    assert np.abs(soft[0].cpu().numpy() - ref[0]).max() <= 2e-5 + tol
    assert np.abs(soft[1].cpu().numpy() / ref[1] - 1).max() <= 1e-4
