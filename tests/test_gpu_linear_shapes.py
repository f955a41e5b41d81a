"""The linear gradient kernel at the edges of its launch shapes.

Its shape follows the row length (lanes, waves and 16-byte chunks of a row), and
its blocks take equal runs of the evaluated rows whatever the partitions, so the
cases are row lengths on both sides of every class in partitions so short that most
blocks have no whole iteration of rows, every class in runs of dozens of iterations
that cross partitions, and few, many and very short partitions.  One step at lr = 1
gives w = w0 - ghat, compared with the same mean gradient in float64 within the fp32
bar (1e-5 normwise).
"""

import ctypes

import numpy as np
import pytest
import torch

import paper_2607_20739_amd as P

from _parity import FP32_TOL, normwise_error

pytestmark = pytest.mark.gpu

# Largest 16-byte chunk count of each class of row lengths.
CLASSES = [1, 2, 4, 6, 8, 12, 16, 32, 48, 56, 64, 96, 112, 128, 192, 224, 256, 320, 384, 512, 640, 768, 896,
           1024, 1280, 1536, 2048, 2560, 3072, 4096, 5120, 6144, 7168, 8192]
LENGTHS = sorted({d for c in CLASSES for d in (4 * c - 3, 4 * c - 1, 4 * c, 4 * c + 1, 4 * c + 4)
                  if d <= 8192 or (d % 4 == 0 and d <= 32768)} | {2, 3})


def _announce(what):
    print("\n[gpu case] " + what, flush=True)


def _mean_gradient(model, X, y, w0):
    X, y, w0 = X.double(), y.double(), w0.double()
    z = X @ w0
    slope = (torch.sigmoid(z) if model == "logistic" else z) - y
    return (X.t() @ slope / X.shape[0]).cpu().numpy()


def _one_step(scheme, model, n, c, X, y, w0, pipelined=True, steps=1):
    sess = P.PGCSession(scheme, n, c, model, X.shape[0], X.shape[1], pipelined=pipelined)
    try:
        w = w0.clone()
        for _ in range(steps):
            sess.step(X, y, w, np.zeros(n, np.uint8), 1.0)
            ghat = sess.decoded()
        torch.cuda.synchronize()
        return ghat, w
    finally:
        sess.close()


@pytest.mark.parametrize("chunk", range(0, len(LENGTHS), 17))
def test_row_lengths_around_every_class(chunk):
    for i, d in enumerate(LENGTHS[chunk:chunk + 17]):
        n, m = ((7, 150), (3, 333), (16, 75))[i % 3]
        model = ("logistic", "lsq")[i % 2]
        _announce("d=%d n=%d m=%d %s" % (d, n, m, model))
        g = torch.Generator(device="cuda")
        g.manual_seed(d)
        X = torch.randn(n * m, d, generator=g, device="cuda")
        y = torch.randint(2, (n * m,), generator=g, device="cuda").float()
        w0 = 0.5 * torch.randn(d, generator=g, device="cuda") / d ** 0.5
        ghat, w = _one_step("FR", model, n, 1, X, y, w0)
        ref = _mean_gradient(model, X, y, w0)
        assert normwise_error(ghat.cpu().numpy(), ref) <= FP32_TOL, d
        assert normwise_error(w.cpu().numpy(), w0.double().cpu().numpy() - ref) <= FP32_TOL, d


@pytest.mark.parametrize("n,m", [(1, 1), (1, 4099), (2, 15), (5, 17), (12, 8191), (31, 3), (64, 16), (100, 129),
                                 (200, 21), (255, 33), (256, 1), (256, 257)])
@pytest.mark.parametrize("d", [20, 1001, 2052, 10240])
def test_blocks_that_cross_partitions(n, m, d):
    """Every ring slot holds its own partition's gradient, whatever blocks its rows fell to."""
    _announce("n=%d m=%d d=%d" % (n, m, d))
    m = min(m, max(1, (1 << 27) // (n * d)))
    g = torch.Generator(device="cuda")
    g.manual_seed(n * m)
    X = torch.randn(n * m, d, generator=g, device="cuda")
    y = torch.randn(n * m, generator=g, device="cuda")
    w = torch.zeros(d, device="cuda")
    sess = P.PGCSession("IS_SGD", n, 1, "lsq", n * m, d)
    try:
        sess.step(X, y, w, np.zeros(n, np.uint8), 0.0)
        for k in sorted({0, 1 % n, n // 2, n - 1}):
            rows = slice(k * m, (k + 1) * m)
            ref = _mean_gradient("lsq", X[rows], y[rows], w)
            assert normwise_error(sess.ring(k, 0).cpu().numpy(), ref) <= FP32_TOL, k
    finally:
        sess.close()


def _partials(n, m, d):
    """Partial sums (32 bits) of a step that evaluates n partitions."""
    size_of = P.lib()["_ZN3pgc21linear_partials_bytesEPK7pgc_ctx"]   # size_t (const pgc_ctx*)
    size_of.restype, size_of.argtypes = ctypes.c_size_t, [ctypes.c_void_p]
    ctx = P.pgc_init("IS_SGD", n, 1, d)
    try:
        P.pgc_configure(ctx, "lsq", n * m, d)
        return size_of(ctx) / (4 * d)
    finally:
        P.pgc_destroy(ctx)


@pytest.mark.parametrize("first", range(0, len(CLASSES) + 1, 5))
def test_every_class_in_long_runs_that_cross_partitions(first):
    """Runs from which blocks cross partition ends have at least four iterations and twelve rows;
    here nine times as many, and some more rows: whole iterations from a scattered start round to
    it, sums moved to LDS several times (every 16 rows of a lane at most), a remainder, and blocks
    with rows of two partitions."""
    for c in ([0] + CLASSES)[first:first + 5]:
        n, d = 9, 3 if c == 0 else 4 * c if c == 1 or 4 * c > 8192 else 4 * c - 1
        m = 16   # blocks within the partitions leave a multiple of n partials
        while _partials(n, m, d) not in [blocks + n - 1 for blocks in (256, 512, 768, 1024)]:
            m = m * 5 // 4 + 1
            assert m < 1 << 20
        m = 9 * m + 5
        _announce("long runs d=%d n=%d m=%d, %d partials" % (d, n, m, _partials(n, m, d)))
        assert (_partials(n, m, d) - n + 1) % 256 == 0
        g = torch.Generator(device="cuda")
        g.manual_seed(d)
        X = torch.randn(n * m, d, generator=g, device="cuda")
        y = torch.randn(n * m, generator=g, device="cuda")
        w = torch.randn(d, generator=g, device="cuda") / d ** 0.5
        sess = P.PGCSession("IS_SGD", n, 1, "lsq", n * m, d)
        try:
            sess.step(X, y, w, np.zeros(n, np.uint8), 0.0)
            for k in (0, 3, n - 1):
                rows = slice(k * m, (k + 1) * m)
                ref = _mean_gradient("lsq", X[rows], y[rows], w)
                assert normwise_error(sess.ring(k, 0).cpu().numpy(), ref) <= FP32_TOL, (d, k)
        finally:
            sess.close()


# n, m: with 20,000 features a block takes at least a row, so min(256 / n, m) partials each.
FOLDS = [(1, m) for m in (1, 2, 3, 4, 5, 7, 8, 9, 10, 12, 13, 31, 32, 33, 36, 39, 40, 71, 256)]
FOLDS += [(3, 40), (17, 5), (40, 3), (64, 4), (60, 8), (64, 1), (85, 2), (128, 3), (130, 3), (256, 2)]


@pytest.mark.parametrize("n,m", FOLDS)
def test_folds_of_any_number_of_partials(n, m):
    """Every remainder of the fold's batches of loads, and one to many rounds of its threads."""
    d = 20000
    _announce("fold n=%d m=%d d=%d" % (n, m, d))
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 1000 + m)
    X = torch.randn(n * m, d, generator=g, device="cuda")
    y = torch.randn(n * m, generator=g, device="cuda")
    w = torch.zeros(d, device="cuda")
    sess = P.PGCSession("CR", n, min(n, 2), "lsq", n * m, d)
    try:
        sess.step(X, y, w, np.zeros(n, np.uint8), 0.0)
        for k in sorted({0, n // 3, n - 1}):
            rows = slice(k * m, (k + 1) * m)
            ref = _mean_gradient("lsq", X[rows], y[rows], w)
            for slot in range(min(n, 2)):
                assert normwise_error(sess.ring((k - slot) % n, slot).cpu().numpy(), ref) <= FP32_TOL, (k, slot)
    finally:
        sess.close()


@pytest.mark.parametrize("n,m", [(4, 1024), (4, 257), (16, 300)])
@pytest.mark.parametrize("d", [16, 20, 64, 100, 128])
def test_short_runs_of_narrow_rows_lose_no_more_than_sums_of_16_rows(n, m, d):
    """Narrow rows share a wave, so a block takes hundreds of rows at once.  The gradient may be off
    by no more than 32-bit sums of 16 rows (two chains of 8) joined in 64 bits make it.  From w = 0
    the slopes are +-1/2, so every term is exact and the error is the sums' alone; it is compared
    over 24 draws, whose root mean square varies by 5% at 16 columns."""
    _announce("precision n=%d m=%d d=%d" % (n, m, d))
    mine, chains = [], []
    for seed in range(24):
        g = torch.Generator().manual_seed(seed)
        X = torch.randn(n * m, d, generator=g)
        y = torch.bernoulli(torch.sigmoid(X @ (torch.randn(d, generator=g) / d ** 0.5)), generator=g)
        sess = P.PGCSession("IS_SGD", n, 1, "logistic", n * m, d)
        try:
            sess.step(X.cuda(), y.cuda(), torch.zeros(d, device="cuda"), np.zeros(n, np.uint8), 0.1)
            got = sess.ring(1, 0).cpu().numpy().astype(np.float64)
        finally:
            sess.close()
        terms = ((0.5 - y)[:, None] * X)[m:2 * m].numpy()
        ref = terms.astype(np.float64).mean(axis=0)
        terms = np.concatenate([terms, np.zeros((-m % 16, d), np.float32)]).reshape(-1, 2, 8, d)
        sums = terms[:, :, 0]
        for i in range(1, 8):
            sums = sums + terms[:, :, i]
        sums = (sums[:, 0] + sums[:, 1]).astype(np.float64).sum(axis=0) * (1.0 / m)
        mine.append(normwise_error(got, ref))
        chains.append(normwise_error(sums.astype(np.float32), ref))
    mine, chains = np.sqrt(np.mean(np.square(mine))), np.sqrt(np.mean(np.square(chains)))
    print("  error %.3g, of sums of 16 rows %.3g" % (mine, chains), flush=True)
    assert mine <= chains


def test_long_runs_of_the_longest_rows_lose_no_more_than_sums_of_16_rows():
    """Blocks of the longest rows take some 60 of them.  As above, against chains of 16 rows."""
    n, m, d = 16, 1000, 20000
    _announce("precision n=%d m=%d d=%d" % (n, m, d))
    mine, chains = [], []
    for seed in range(3):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        X = torch.randn(n * m, d, generator=g, device="cuda")
        y = torch.randint(2, (n * m,), generator=g, device="cuda").float()
        sess = P.PGCSession("IS_SGD", n, 1, "logistic", n * m, d)
        try:
            sess.step(X, y, torch.zeros(d, device="cuda"), np.zeros(n, np.uint8), 0.1)
            got = sess.ring(1, 0).double()
        finally:
            sess.close()
        terms = (0.5 - y[m:2 * m])[:, None] * X[m:2 * m]
        ref = terms.double().mean(dim=0)
        terms = torch.nn.functional.pad(terms, (0, 0, 0, -m % 16)).view(-1, 16, d)
        sums = terms[:, 0]
        for i in range(1, 16):
            sums = sums + terms[:, i]
        sums = (sums.double().sum(dim=0) * (1.0 / m)).float().double()
        mine.append(float((got - ref).norm() / ref.norm()))
        chains.append(float((sums - ref).norm() / ref.norm()))
    mine, chains = np.sqrt(np.mean(np.square(mine))), np.sqrt(np.mean(np.square(chains)))
    print("  error %.3g, of sums of 16 rows %.3g" % (mine, chains), flush=True)
    assert mine <= chains


def test_any_base_address_gives_the_same_bits():
    n, m, d = 6, 211, 1000
    _announce("X and w at every float offset, d=%d" % d)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X = torch.randn(n * m, d, generator=g, device="cuda")
    y = torch.randint(2, (n * m,), generator=g, device="cuda").float()
    w0 = torch.randn(d, generator=g, device="cuda") / d ** 0.5
    ref = None
    for off in range(4):
        Xo = torch.empty(n * m * d + 4, device="cuda")[off:off + n * m * d].view(n * m, d).copy_(X)
        wo = torch.empty(d + 4, device="cuda")[off:off + d].copy_(w0)
        sess = P.PGCSession("FR", n, 3, "logistic", n * m, d)
        try:
            for _ in range(3):
                sess.step(Xo, y, wo, np.zeros(n, np.uint8), 0.1)
            got = wo.clone()
        finally:
            sess.close()
        ref = got if ref is None else ref
        assert torch.equal(got, ref), off


@pytest.mark.parametrize("d", [7, 69, 1001, 4099])
def test_infinite_features_reach_only_what_they_touch(d):
    """An infinite feature makes its row's z infinite (the sigmoid's limit), and its own column
    infinite; the floats the last chunk shares with another lane add nothing of their own."""
    n, m = 2, 40
    _announce("infinite feature, d=%d" % d)
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    X = torch.randn(n * m, d, generator=g, device="cuda")
    y = torch.zeros(n * m, device="cuda")
    w0 = torch.ones(d, device="cuda") / d
    for col in (0, d - 5, d - 4, d - 3, d - 1):
        Xi = X.clone()
        Xi[3, col] = float("inf")
        ghat, _ = _one_step("FR", "logistic", n, 1, Xi, y, w0)
        ref = _mean_gradient("logistic", Xi, y, w0)
        got = ghat.cpu().numpy()
        fine = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), fine) and fine.sum() == d - 1, col
        assert normwise_error(got[fine], ref[fine]) <= FP32_TOL, col


@pytest.mark.parametrize("d", [100, 4096, 16388, 32768])
def test_an_infinite_sum_stays_infinite(d):
    """Sums that overflow 32 bits early in a run of several moves to LDS: an infinite sum gives back
    no rounding (that would be NaN), so its column ends infinite and the others as they were."""
    n, m = 1, (1 << 26) // d
    _announce("infinite sum, d=%d m=%d" % (d, m))
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    X = torch.randn(n * m, d, generator=g, device="cuda")
    y = torch.full((n * m,), 2.0, device="cuda")
    w0 = torch.zeros(d, device="cuda")
    X[0, 5] = X[m // 2, d - 2] = 0.0
    plain, _ = _one_step("FR", "lsq", n, 1, X, y, w0)
    X[0, 5], X[m // 2, d - 2] = 3e38, -3e38   # slope -2
    got, _ = _one_step("FR", "lsq", n, 1, X, y, w0)
    keep = torch.ones(d, dtype=torch.bool, device="cuda")
    keep[5] = keep[d - 2] = False
    assert got[5] == -float("inf") and got[d - 2] == float("inf")
    assert torch.equal(got[keep], plain[keep])
