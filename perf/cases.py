"""The calls that the performance of the PGC step is measured on.

A case is one training step through PGCSession: the gradients of the evaluated
partitions, the ring write, the encode, the masked decode and the update, on
data that stays in GPU memory.  The pipeline is filled (t = 0) beforehand, as
it is for all but the first step of a run; gradient coding (pipelined = False)
evaluates every slot at every step, as the fill does.
"""

import math

import numpy as np
import torch

import paper_2607_20739_amd as P

MASKS = 64                 # straggler masks a state cycles through
CHUNK = 1 << 27            # feature values the 64-bit evaluation widens at a time
CODE_SEED = 2              # seed of the real-valued code's random matrix


def listed():
    return [
        # The smallest call of the repository: 2,048 rows of 64 features per step, bound by
        # launches and latency (a small tabular problem, many steps per second).
        linear("fr_logistic_d64", "FR", "logistic", n=4, c=2, m=1024, d=64, lr=0.1),
        # One-against-rest logistic regression over 60,000 images of 28 x 28, ignoring stragglers:
        # a comparison system, on features that still fit the last cache.
        linear("is_sgd_logistic_d784", "IS_SGD", "logistic", n=12, c=1, m=5000, d=784),
        # Tables come with any number of columns: rows that start at no particular alignment, and
        # partitions whose row count divides by nothing.
        linear("cr_logistic_odd_d1001", "CR", "logistic", n=12, c=4, m=8191, d=1001),
        # The naive real-valued code on least squares, 1 GiB of features per step.
        linear("crreal_lsq_d1024", "CR_REAL", "lsq", n=8, c=3, m=32768, d=1024, lr=0.001),
        # Gradient coding with the real-valued code (every slot evaluated at every step): the
        # other comparison system, 12 workers of 65,536 rows.
        linear("gc_lsq_d1024", "CR_REAL", "lsq", n=12, c=3, m=65536, d=1024, pipelined=False),
        # Wide rows (bag-of-words features), full-batch gradient descent without repetition.
        linear("dgd_lsq_d20000", "FR", "lsq", n=16, c=1, m=1000, d=20000),
        # PGC-FR on 16 GiB of features with every tenth column ten times larger; a step reads a
        # quarter of them.
        linear("fr_logistic_d4096", "FR", "logistic", n=32, c=4, m=32768, d=4096, scale_every=10),
        # PGC-CR with many workers and a deep pipeline, 16 GiB of features read by every step.
        linear("cr_logistic_d8192", "CR", "logistic", n=128, c=8, m=4096, d=8192),
        # The smallest network: latency and the number of launches.
        mlp("cr_mlp_small", "CR", n=4, c=2, m=64, d=64, hidden=256, classes=10),
        # The 784 -> 1024 -> 10 network on small batches, 256 rows per partition: the weights and
        # their gradients outweigh the rows.
        mlp("cr_mlp_256_rows", "CR", n=64, c=4, m=256, d=784, hidden=1024, classes=10),
        # The same images split over 12 workers, PGC-FR: four partitions of 5,000 rows per step
        # and a network half as wide.
        mlp("fr_mlp_5000_rows", "FR", n=12, c=3, m=5000, d=784, hidden=512, classes=10),
        # The same network over a million rows: matrix products all the way.
        mlp("cr_mlp_16384_rows", "CR", n=64, c=4, m=16384, d=784, hidden=1024, classes=10),
    ]


def linear(name, scheme, model, n, c, m, d, lr=0.01, scale_every=0, pipelined=True):
    return dict(name=name, scheme=scheme, model=model, n=n, c=c, m=m, d=d, hidden=0, classes=0, lr=lr,
                scale_every=scale_every, pipelined=pipelined)


def mlp(name, scheme, n, c, m, d, hidden, classes, lr=0.01, pipelined=True):
    return dict(name=name, scheme=scheme, model="mlp", n=n, c=c, m=m, d=d, hidden=hidden, classes=classes, lr=lr,
                scale_every=0, pipelined=pipelined)


def draw(rng):
    """A case of the listed ones' ranges: features, rows, workers and repetition over their
    logarithms, every scheme, pipelined or not, odd sizes included."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    scheme = rng.choice(["FR", "FR", "CR", "CR", "CR_REAL", "IS_SGD"])
    c = 1 if scheme == "IS_SGD" else rng.randint(2, 3) if scheme == "CR_REAL" else rng.choice([1, 2, 3, 4, 6, 8])
    if scheme == "FR":
        n = c * log_int(1, 128 // c)
    elif scheme == "CR_REAL":
        n = rng.randint(max(4, c), 12)
    else:
        n = log_int(max(4, c), 128)
    pipelined = rng.random() < 0.8
    if rng.random() < 0.35:
        d = 8 * log_int(2, 400)
        hidden = 256 * rng.randint(1, 4)
        rows = log_int(64, min(400000, int(6e11 / (4 * d * hidden))))
        return dict(mlp("", scheme, n=n, c=c, m=max(16, rows // n), d=d, hidden=hidden, classes=rng.randint(2, 16),
                        pipelined=pipelined), name="drawn")
    d = log_int(16, 32768)
    if d > 8192 or rng.random() < 0.5:
        d -= d % 4          # wider rows than 8192 come in multiples of four
    values = log_int(1 << 16, 1 << 30)    # features in all, up to 4 GiB
    m = max(16, values // (n * d))
    model = "lsq" if scheme == "CR_REAL" else rng.choice(["logistic", "logistic", "lsq"])
    lr = 0.001 if scheme == "CR_REAL" else 0.01
    if model == "lsq":      # below the stability limit of few rows with many features
        lr = min(lr, 0.1 / (1 + math.sqrt(d / (m * n))) ** 2)
    return dict(linear("", scheme, model, n=n, c=c, m=m, d=d, lr=lr, pipelined=pipelined), name="drawn")


def inputs(case, seed):
    """Features, labels, first weights and straggler masks, from the seed alone."""
    N, d = case["n"] * case["m"], case["d"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["model"] == "mlp":
        hidden, classes = case["hidden"], case["classes"]
        X = torch.empty(N, d, dtype=torch.bfloat16, device="cuda").uniform_(0.0, 1.0, generator=g)
        y = torch.randint(classes, (N,), generator=g, device="cuda", dtype=torch.int32)
        W1 = torch.randn(d * hidden, generator=g, device="cuda") * math.sqrt(2.0 / d)
        W2 = torch.randn(hidden * classes, generator=g, device="cuda") * math.sqrt(2.0 / hidden)
        w = torch.cat([W1, torch.zeros(hidden, device="cuda"), W2, torch.zeros(classes, device="cuda")])
    else:
        X = torch.randn(N, d, generator=g, device="cuda")
        if case["scale_every"]:
            X[:, ::case["scale_every"]] *= 10.0
        planted = torch.randn(d, generator=g, device="cuda") / math.sqrt(d)
        z = torch.cat([rows @ planted for rows in X.split(1 << 16)])
        if case["model"] == "logistic":
            y = torch.bernoulli(torch.sigmoid(z), generator=g)
        else:
            y = z + 0.1 * torch.randn(N, generator=g, device="cuda")
        w = torch.zeros(d, device="cuda")
    # Up to c - 1 stragglers (IS_SGD ignores any; a tenth of the workers here).
    draws = np.random.RandomState(seed)
    most = case["n"] // 10 if case["scheme"] == "IS_SGD" else case["c"] - 1
    masks = np.zeros((MASKS, case["n"]), dtype=np.uint8)
    for row in masks:
        row[draws.permutation(case["n"])[:draws.randint(most + 1)]] = 1
    return X, y, w, masks


def prepare(case, seed):
    X, y, w, masks = inputs(case, seed)
    session = P.PGCSession(case["scheme"], case["n"], case["c"], case["model"], X.shape[0], case["d"],
                           hidden=case["hidden"], classes=case["classes"], code_seed=CODE_SEED,
                           pipelined=case["pipelined"])
    session.step(X, y, w, masks[0], case["lr"])    # fills the pipeline
    return {"session": session, "X": X, "y": y, "w": w, "masks": masks, "lr": case["lr"], "t": 1,
            "keep": case["model"] == "mlp"}


def run(state):
    session, w = state["session"], state["w"]
    mask = state["masks"][state["t"] % MASKS]
    state["t"] += 1
    session.step(state["X"], state["y"], w, mask, state["lr"])
    # A network's weights hardly move in one step, so its gradient is read as well; the linear
    # models start from zero, and their weights are the sum of the steps taken.
    return {"w": w, "gradient": session.decoded()} if state["keep"] else {"w": w}


def evaluated(case):
    """Partitions a step evaluates."""
    return case["n"] // case["c"] if case["scheme"] == "FR" and case["pipelined"] else case["n"]


def work(case):
    n, c, d, hidden, classes = case["n"], case["c"], case["d"], case["hidden"], case["classes"]
    fr = case["scheme"] == "FR"
    rows = evaluated(case) * case["m"]
    if case["model"] == "mlp":
        q = d * hidden + hidden + hidden * classes + classes
        flops = rows * (4.0 * d * hidden + 6.0 * hidden * classes)
        per_row = 2 * d + 4
    else:
        q, flops, per_row = d, 4.0 * rows * d, 4 * d + 4
    # Each worker's slots (FR: each partition's copy) are either written afresh or read; then the
    # coded words (FR: one per group), the decoded gradient, and w read and written.
    slots = n if fr else n * c
    coded = n // c if fr else n
    return {"bytes": rows * per_row + 4.0 * q * (slots + coded + 1 + 2), "flops": flops}


def tolerance(case):
    if case["model"] == "mlp":
        # H, dZ2 and dZ1 in bf16 between 32-bit sums: 1e-3 off at most with few rows; the gradient is
        # a mean over rows, in which their rounding averages out (1.5e-5 over a million rows).
        return {"rel": 5e-3}
    # The real-valued code's decode cancels terms many times larger than its result.
    return {"rel": 4e-5 if case["scheme"] == "CR_REAL" else 1e-5}


# The same step in 64 bits.

def exact(case, seed):
    X, y, w, masks = inputs(case, seed)
    w = w.double()
    n, c, fr = case["n"], case["c"], case["scheme"] == "FR"
    B = real_code(case) if case["scheme"] == "CR_REAL" else None
    copies = {}                       # (partition, slot) -> gradient; FR keeps one copy, slot 0
    ghat = None
    for t in (0, 1):
        every = t == 0 or not case["pipelined"]
        # At t = 1 the pipeline evaluates slot 0: FR partition j c of each group j, CR all.
        for k in range(n):
            if every or not fr or k % c == 0:
                g = gradient(case, X, y, w, k)
                for slot in range(c if every and not fr else 1):
                    copies[k, slot] = g
        alive = [i for i in range(n) if not masks[t % MASKS][i]]
        ghat = torch.zeros_like(w)
        if fr:
            for k in range(n):
                ghat += copies[k, 0] / n
        elif B is not None:
            weights = np.linalg.pinv(B[alive].T) @ np.ones(n)
            for a, j in zip(weights, alive):
                for o in range(c):
                    ghat += float(a * B[j, (j + o) % n] / n) * copies[(j + o) % n, o]
        else:
            for j in alive:
                for o in range(c):
                    ghat += copies[(j + o) % n, o] / (len(alive) * c)
        w = w - float(np.float32(case["lr"])) * ghat
        if t == 0:
            w = w.float().double()    # the caller's vector is 32 bits wide
    return {"w": w, "gradient": ghat} if case["model"] == "mlp" else {"w": w}


def gradient(case, X, y, w, k):
    """Mean gradient of partition k's rows at w."""
    m, d = case["m"], case["d"]
    total = torch.zeros_like(w)
    step = max(1, CHUNK // max(d, case["hidden"]))
    for r in range(k * m, (k + 1) * m, step):
        rows = slice(r, min(r + step, (k + 1) * m))
        x, label = X[rows].double(), y[rows]
        if case["model"] == "mlp":
            total += network_gradient(case, x, label, w)
        else:
            z = x @ w
            slope = (torch.sigmoid(z) if case["model"] == "logistic" else z) - label.double()
            total += x.t() @ slope
    return total / m


def network_gradient(case, x, label, w):
    d, hidden, classes = case["d"], case["hidden"], case["classes"]
    at = d * hidden
    # The layers use the weight matrices rounded to bf16.
    W1 = w[:at].float().bfloat16().double().view(d, hidden)
    b1 = w[at:at + hidden]
    W2 = w[at + hidden:at + hidden + hidden * classes].float().bfloat16().double().view(hidden, classes)
    b2 = w[-classes:]
    h = torch.relu(x @ W1 + b1)
    dz2 = torch.softmax(h @ W2 + b2, dim=1)
    dz2[torch.arange(len(label), device=dz2.device), label.long()] -= 1.0
    dz1 = (dz2 @ W2.t()) * (h > 0)
    return torch.cat([(x.t() @ dz1).reshape(-1), dz1.sum(0), (h.t() @ dz2).reshape(-1), dz2.sum(0)])


def real_code(case):
    """The n x n real-valued cyclic code: row j is 1 at j, supported on {j .. j + c - 1} mod n, and
    in the null space of a random matrix whose rows sum to zero (SplitMix64's draws in [-1, 1))."""
    n, s, wide = case["n"], case["c"] - 1, (1 << 64) - 1

    def uniform(index):
        z = (CODE_SEED + (index + 1) * 0x9E3779B97F4A7C15) & wide
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & wide
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & wide
        return 2.0 * (((z ^ (z >> 31)) >> 11) * 2.0 ** -53) - 1.0

    H = np.array([[uniform(a * n + k) for k in range(n)] for a in range(s)]).reshape(s, n)
    H[:, -1] = -H[:, :-1].sum(axis=1)
    B = np.eye(n)
    for j in range(n):
        others = [(j + o) % n for o in range(1, s + 1)]
        B[j, others] = np.linalg.solve(H[:, others], -H[:, j])
    return B
