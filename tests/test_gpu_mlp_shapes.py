"""The MLP gradient over the shapes at which its kernels change course: every row tile of the
rows kernel at each hidden width (few, some and many rows), runs of tiles that cross
partitions, tiles past a partition's rows, one and two K slices, and K loops long enough that
every slot of the ring of W1 slices is used again.

Each part of every partition's gradient (dW1, db1, dW2, db2) is compared with the fp64 oracle
on the ring after the first step.  H, dZ2 and dZ1 are rounded to bf16 (2^-9 of each term at
most), so a part is off by a few 2^-9 of its largest entry where few rows are summed: the bf16
bar of 2e-2 covers that.
"""

import ctypes

import numpy as np
import pytest
import torch

import paper_2607_20739_amd as P
from oracle import pgc_oracle as O

from _parity import normwise_error

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2

# n, m, d_in, hidden, classes
SHAPES = [
    (4, 100, 64, 256, 10), (4, 2000, 32, 256, 4), (4, 3000, 8, 256, 3), (3, 20000, 40, 256, 16),
    (3, 700, 264, 512, 5), (4, 3400, 200, 512, 16), (3, 22000, 72, 512, 10), (4, 8100, 72, 512, 10),
    (3, 65, 24, 768, 2), (4, 3400, 96, 768, 9), (4, 4400, 96, 768, 9), (3, 15990, 40, 768, 4),
    (4, 1000, 32, 1024, 13), (4, 3400, 784, 1024, 10), (4, 5000, 72, 1024, 7),
    (3, 16100, 104, 1024, 10),
    (5, 1, 16, 1024, 2), (65, 33, 48, 256, 7),
]


class _Grid(ctypes.Structure):
    _fields_ = [("tiles_per_part", ctypes.c_int64), ("blocks", ctypes.c_int32), ("runs", ctypes.c_int32),
                ("shape", ctypes.c_int)]


def _rows_grid(n, m, d, hidden):
    """The rows kernel's grid: MlpRowsGrid pgc::mlp_rows_grid(m_pad, n_eval, kslices, hidden)."""
    rule = P.lib()["_ZN3pgc13mlp_rows_gridEliii"]
    rule.restype, rule.argtypes = _Grid, [ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32]
    return rule((m + 63) // 64 * 64, n, (d + 31) // 32, hidden)


def _rows_for(n, d, hidden, shape, rounds):
    """The fewest rows per partition (of some) whose tile is the shape-th and whose blocks have at
    least so many tiles."""
    for m in list(range(43, 4000, 60)) + list(range(4003, 24000, 500)):
        g = _rows_grid(n, m, d, hidden)
        if g.shape == shape and g.tiles_per_part * n > (rounds - 1) * g.blocks:
            return m
    return None


@pytest.mark.parametrize("d", [296, 328])   # 10 and 11 K slices; the ring has 4, 3 or 2 slots
@pytest.mark.parametrize("shape", range(4))
@pytest.mark.parametrize("hidden", [256, 512, 768, 1024])
def test_every_row_tile_in_long_k_loops(hidden, shape, d):
    """The ring's loads are ordered by counts of loads in flight, which apply from as many slices on
    as the ring has and reuse a slot from one more; a wrong one reads a stale slice of W1."""
    one, several = _rows_for(5, d, hidden, shape, 1), _rows_for(3, d, hidden, shape, 2)
    assert one is not None and (several is not None or shape > 1)   # low tiles are for few rows
    for n, m in ((5, one), (3, several)):
        if m is None:
            continue
        assert _rows_grid(n, m, d, hidden).shape == shape
        test_partition_gradients_match_the_oracle(n, m, d, hidden, 2 + (m + shape) % 15)


@pytest.mark.parametrize("n,m,d,hidden,classes", SHAPES)
def test_partition_gradients_match_the_oracle(n, m, d, hidden, classes):
    print("\n[gpu case] MLP n=%d m=%d %d-%d-%d" % (n, m, d, hidden, classes), flush=True)
    q = d * hidden + hidden + hidden * classes + classes
    g = torch.Generator().manual_seed(n + m + d + hidden)
    X = torch.rand(n * m, d, generator=g).bfloat16()
    y = torch.randint(classes, (n * m,), generator=g, dtype=torch.int32)
    w = torch.randn(q, generator=g) * 0.1
    sess = P.PGCSession("CR", n, 2, "mlp", n * m, d, hidden=hidden, classes=classes)
    try:
        wd = w.cuda()
        sess.step(X.cuda(), y.cuda(), wd, np.zeros(n, np.uint8), 0.0)
        assert torch.equal(wd.cpu(), w)
        cuts = np.cumsum([d * hidden, hidden, hidden * classes])
        for k in sorted({0, n // 2, n - 1}):
            ref = O.partition_gradient(O.MLP, X[k * m:(k + 1) * m].double().numpy(), y[k * m:(k + 1) * m].numpy(),
                                       w.double().numpy(), (d, hidden, classes))
            got = sess.ring(k, 0).cpu().numpy()
            errs = [normwise_error(a, b) for a, b in zip(np.split(got, cuts), np.split(ref, cuts))]
            print("  partition %d: dW1 %.2g db1 %.2g dW2 %.2g db2 %.2g" % ((k,) + tuple(errs)), flush=True)
            assert max(errs) <= BF16_TOL
    finally:
        sess.close()


@pytest.mark.parametrize("n,m,hidden", [(1, 1 << 20, 256), (1, 1 << 20, 1024), (2, (1 << 19) + 16 * 333, 768)])
def test_sums_of_a_million_rows_lose_no_more_than_sums_of_1024(n, m, hidden):
    """dW2 is a sum over rows whose terms are exact here: W1 copies features into the hidden layer,
    W2 = 0 makes the softmax 1/2.  It may be off by no more than 32-bit sums of 1,024 rows, 16 at a
    time, joined in 64 bits (random labels, so the sums wander; 64 columns of 4 draws)."""
    d, classes = 64, 2
    print("\n[gpu case] MLP precision n=%d m=%d hidden=%d" % (n, m, hidden), flush=True)
    mine, chains = [], []
    for seed in range(4):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        X = torch.rand(n * m, d, generator=g, device="cuda").bfloat16()
        y = torch.randint(2, (n * m,), generator=g, device="cuda", dtype=torch.int32)
        W1 = torch.zeros(d, hidden, device="cuda")
        W1[torch.arange(hidden) % d, torch.arange(hidden)] = 1.0
        w = torch.cat([W1.reshape(-1), torch.zeros(hidden + hidden * classes + classes, device="cuda")])
        sess = P.PGCSession("IS_SGD", n, 1, "mlp", n * m, d, hidden=hidden, classes=classes)
        try:
            sess.step(X, y, w, np.zeros(n, np.uint8), 0.0)
            got = sess.ring(n - 1, 0)[d * hidden + hidden:-classes].view(hidden, classes)[:d, 0].double()
        finally:
            sess.close()
        dz = (0.5 - (y[(n - 1) * m:] == 0).double()) * float(torch.tensor(1.0 / m))
        terms = X[(n - 1) * m:].double() * dz.bfloat16().double()[:, None]
        ref = terms.sum(dim=0)
        steps = torch.nn.functional.pad(terms, (0, 0, 0, -m % 1024)).view(-1, 64, 16, d).sum(dim=2).float()
        sums = steps[:, 0]
        for i in range(1, 64):
            sums = sums + steps[:, i]
        sums = sums.double().sum(dim=0).float().double()
        mine.append(float((got - ref).norm() / ref.norm()))
        chains.append(float((sums - ref).norm() / ref.norm()))
        del X, terms, steps
    mine, chains = np.sqrt(np.mean(np.square(mine))), np.sqrt(np.mean(np.square(chains)))
    print("  error %.3g, of sums of 1,024 rows %.3g" % (mine, chains), flush=True)
    assert mine <= chains
