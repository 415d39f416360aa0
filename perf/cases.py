"""The calls whose speed matters to a program that uses this library, with inputs of the sizes that occur.

Every case goes through the public Python entry points (paper_2106_05203_amd.binding).  The kinds:

  topk      ef21_topk on a batch of rows: the stand-alone compressor
  steps     an experiment on a dense logistic regression problem: set_state, T times step(), get_state
  grad      EF21.local_grad of a dense problem, either loss, all rows or a minibatch (Algorithm 5)
  csr       EF21.local_grad of a sparse problem
  update    one step() with supplied gradients (a network's flat gradients) and the new model:
            algorithm "ef21" (Algorithm 2, either loop order), "plus" (Algorithm 3) or "ef" (Algorithm 4)
  stepsize  EF21.theory_stepsize, which a program calls once per problem before its first step

Inputs are drawn on the GPU from the seed alone.  Where consecutive calls of a real program get fresh data (the
gradients of `update`), a state holds a pool of independent draws and each pass takes the next one.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_05203_amd import binding

LAM = 0.1      # regulariser of the logistic problems, the paper's value
DEV = "cuda"


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest problem of the test configurations (4 workers, 1000 rows in all, Top-1): bound by latency
        dict(name="steps_small", kind="steps", n=4, d=100, m=250, k=1, gamma=0.1, steps=20),
        # the shape of the paper's a9a experiment: 20 clients of 1628 rows, 123 features (odd rows), k = 4
        dict(name="steps_a9a", kind="steps", n=20, d=123, m=1628, k=4, gamma=0.5, steps=10),
        # the headline dense problem: 800 MB of rows, whole iterations
        dict(name="steps_large", kind="steps", n=20, d=2000, m=5000, k=20, gamma=0.5, steps=4),
        # the gradient of a problem with many features per row, least squares
        dict(name="grad_wide", kind="grad", n=8, d=12000, m=2000, loss=1, tau=0),
        # a minibatch of an eighth of the rows of the headline problem
        dict(name="grad_minibatch", kind="grad", n=20, d=2000, m=5000, loss=0, tau=625),
        # the headline sparse problem: 100 workers, 10^8 entries, one per cent filled
        dict(name="csr_large", kind="csr", n=100, d=50000, m=2000, nnz=500, ragged=False),
        # the stand-alone compressor on long rows, one per cent kept
        dict(name="topk_long", kind="topk", n=20, d=1000000, k=10000),
        # ... and on many rows of moderate length
        dict(name="topk_mid", kind="topk", n=100, d=50000, k=500),
        # flat network gradients of 8 workers, one per cent kept
        dict(name="update_network", kind="update", algo="ef21", n=8, d=11200000, k=112000, order=0, noise=1.0),
        # EF21+ at the size of ResNet18 with the paper's 5 clients and 5 per cent kept
        dict(name="plus_resnet18", kind="update", algo="plus", n=5, d=11511784, k=575589, order=0, noise=0.3),
        # the original EF on gradients of an odd length
        dict(name="ef_odd", kind="update", algo="ef", n=5, d=1000003, k=50000, order=0, noise=1.0),
        # the stepsize of Theorem 1 for the shape of the paper's w8a experiment
        dict(name="stepsize_w8a", kind="stepsize", n=20, d=300, m=2487, k=4, iterations=100),
    ]


def _log_int(rng, lo, hi):
    """A whole number in [lo, hi], uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["topk", "topk", "steps", "steps", "grad", "grad", "csr", "update", "update", "plus", "ef",
                       "stepsize"])
    if kind == "topk":
        d = _log_int(rng, 100, 10000000)
        n = _log_int(rng, 1, max(1, min(200, 100000000 // d)))
        k = max(1, int(d * math.exp(rng.uniform(math.log(1e-4), math.log(0.1)))))
        return dict(kind="topk", n=n, d=d, k=k)
    if kind in ("steps", "grad", "stepsize"):
        most = 15000000 if kind == "stepsize" else 200000000            # matrix entries
        n = _log_int(rng, 2, 32)
        d = _log_int(rng, 50, {"steps": 3000, "grad": 20000, "stepsize": 1000}[kind])
        m = _log_int(rng, 100, max(100, min(8000, most // (n * d))))
        if kind == "steps":
            k = min(rng.choice([1, 2, 4, 8, 16, 32, 64]), d // 4)
            steps = max(1, min(20, 1000 // (n * k), 800000000 // (n * m * d)))
            return dict(kind="steps", n=n, d=d, m=m, k=k, gamma=0.2, steps=steps)
        if kind == "grad":
            tau = 0 if rng.random() < 0.6 else max(1, m // rng.choice([4, 8, 16]))
            return dict(kind="grad", n=n, d=d, m=m, loss=rng.choice([0, 1]), tau=tau)
        return dict(kind="stepsize", n=n, d=d, m=m, k=max(1, d // 50), iterations=100)
    if kind == "csr":
        d = _log_int(rng, 1000, 200000)
        nnz = _log_int(rng, 5, min(500, d // 20))
        n = _log_int(rng, 2, 100)
        m = _log_int(rng, 100, max(100, min(10000, 100000000 // (n * nnz))))
        n = max(1, min(n, 50000000 // d))                                 # gradients of at most 200 MB
        return dict(kind="csr", n=n, d=d, m=m, nnz=nnz, ragged=rng.random() < 0.5)
    algo = {"update": "ef21"}.get(kind, kind)
    n = _log_int(rng, 2, 32)
    most = 89000000 if algo == "ef21" else 57000000
    d = _log_int(rng, 10000, most // n)
    k = max(2, int(d * math.exp(rng.uniform(math.log(1e-3), math.log(0.06)))))
    return dict(kind="update", algo=algo, n=n, d=d, k=k, order=rng.choice([0, 1]) if algo != "ef" else 0,
                noise=rng.choice([0.1, 1.0]))


# ---------------------------------------------------------------- inputs
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7fffffffffff)
    return g


def _topk_rows(case, seed):
    """N(0,1) rows in which one entry in a hundred is a copy of another with alternating sign: exact ties."""
    n, d = case["n"], case["d"]
    g = _gen(seed, 1)
    v = torch.randn((n, d), device=DEV, generator=g)
    c = d // 100
    if c:
        dst = torch.randint(0, d, (n, c), device=DEV, generator=g)
        src = torch.randint(0, d, (n, c), device=DEV, generator=g)
        sign = torch.ones(c, device=DEV)
        sign[1::2] = -1.0
        for i in range(n):                       # later copies win where a position is drawn twice: keep the first
            at, first = torch.unique(dst[i], return_inverse=True)
            pick = torch.full((at.numel(),), c, device=DEV, dtype=torch.int64)
            pick.scatter_reduce_(0, first, torch.arange(c, device=DEV), "amin")
            v[i, at] = v[i, src[i, pick]] * sign[pick]
    return v


def _dense(case, seed):
    """Rows N(0,1)/sqrt(d); labels sign(A w*) with a tenth flipped, or targets A w* + noise for least squares."""
    n, d, m = case["n"], case["d"], case["m"]
    g = _gen(seed, 2)
    A = torch.randn((n, m, d), device=DEV, generator=g).mul_(1.0 / math.sqrt(d))
    w = torch.randn(d, device=DEV, generator=g)
    z = torch.mv(A.view(n * m, d), w).view(n, m)
    if case.get("loss", 0) == 1:
        y = z + 0.1 * torch.randn((n, m), device=DEV, generator=g)
    else:
        flip = torch.rand((n, m), device=DEV, generator=g) < 0.1
        y = torch.where((z >= 0) ^ flip, 1.0, -1.0)
    x = torch.randn(d, device=DEV, generator=g).mul_(0.1)
    return A, y.float().contiguous(), x


def _batch(case, seed):
    return torch.randint(0, case["m"], (case["n"], case["tau"]), device=DEV, generator=_gen(seed, 3),
                         dtype=torch.int32)


def _csr(case, seed):
    """Rows of `nnz` distinct ascending columns (ragged: a random half to all of them), values U(0,1)."""
    n, d, m, nnz = case["n"], case["d"], case["m"], case["nnz"]
    g = _gen(seed, 4)
    rows = n * m
    # ascending draws with repetition from [0, d - nnz], shifted by their rank: distinct
    col = torch.randint(0, d - nnz + 1, (rows, nnz), device=DEV, generator=g, dtype=torch.int32)
    col = col.sort(dim=1).values.add_(torch.arange(nnz, device=DEV, dtype=torch.int32))
    val = torch.rand((rows, nnz), device=DEV, generator=g)
    if case["ragged"]:
        length = torch.randint(nnz // 2, nnz + 1, (rows,), device=DEV, generator=g)
        keep = torch.arange(nnz, device=DEV)[None, :] < length[:, None]
        col, val = col[keep], val[keep]
    else:
        length = torch.full((rows,), nnz, device=DEV, dtype=torch.int64)
    rowptr = torch.zeros(rows + 1, device=DEV, dtype=torch.int64)
    rowptr[1:] = torch.cumsum(length, 0)
    y = torch.where(torch.rand((n, m), device=DEV, generator=g) < 0.5, 1.0, -1.0)
    x = torch.randn(d, device=DEV, generator=g).mul_(0.1)
    return rowptr, col.reshape(-1).contiguous(), val.reshape(-1).contiguous(), y, x


POOL = 4       # gradient sets that the passes of an `update` case take in turn


def _t3(n, d, g):
    """Student-t with three degrees of freedom, scaled by 1e-3: heavy tails, as flat network gradients have."""
    z = torch.randn((n, d), device=DEV, generator=g)
    chi = torch.zeros((n, d), device=DEV)
    for _ in range(3):
        chi.add_(torch.randn((n, d), device=DEV, generator=g).square_())
    return z.div_(chi.div_(3.0).sqrt_()).mul_(1e-3)


def _gradients(case, seed, count):
    """g_i^0 and `count` gradient sets: worker i's are a fixed part plus fresh noise, whose share goes from
    `noise` (first worker) to 1 (last worker); noise = 1: independent draws."""
    n, d, noise = case["n"], case["d"], case["noise"]
    g = _gen(seed, 5)
    if noise >= 1.0:
        return _t3(n, d, g), [_t3(n, d, g) for _ in range(count)]
    base = _t3(n, d, g)
    share = torch.linspace(noise, 1.0, n, device=DEV)[:, None]
    return base, [(base * (1.0 - share)).add_(_t3(n, d, g).mul_(share)) for _ in range(count)]


GAMMA = 0.01   # learning rate of the `update` cases


def _flags(case):
    order = binding.ORDER_STEP_FIRST if case["order"] else binding.ORDER_GRAD_FIRST
    return {"ef21": order, "plus": order | binding.PLUS, "ef": binding.CLASSIC_EF}[case["algo"]]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "topk":
        return dict(kind=kind, rows=_topk_rows(case, seed), k=case["k"])
    n, d = case["n"], case["d"]
    if kind == "csr":
        rowptr, col, val, y, x = _csr(case, seed)
        h = binding.EF21(n, d, max(1, d // 100), 0.5)
        h.set_problem_csr(rowptr, col, val, y, case["m"], LAM)
        return dict(kind=kind, h=h, x=x, out=torch.empty((n, d), device=DEV))
    if kind == "update":
        g0, pool = _gradients(case, seed, POOL)
        h = binding.EF21(n, d, case["k"], GAMMA)
        if case["algo"] == "ef":
            g0.zero_()                           # Algorithm 4 starts from zero errors
        h.set_state(x=torch.zeros(d, device=DEV), g_i=g0)
        return dict(kind=kind, h=h, pool=pool, at=0, flags=_flags(case))
    A, y, x = _dense(case, seed)
    h = binding.EF21(n, d, case.get("k", max(1, d // 100)), case.get("gamma", 0.5))
    h.set_problem_dense(A, y, 0.0 if case.get("loss", 0) == 1 else LAM)
    h.set_loss(case.get("loss", 0))
    if kind == "steps":
        g_i = h.local_grad(x)
        return dict(kind=kind, h=h, x=x, g_i=g_i, steps=case["steps"])
    if kind == "stepsize":
        return dict(kind=kind, h=h, iterations=case["iterations"])
    if case["tau"]:
        h.set_minibatch(_batch(case, seed))
    return dict(kind=kind, h=h, x=x, out=torch.empty((n, d), device=DEV))


# ---------------------------------------------------------------- one pass
def run(state):
    kind = state["kind"]
    if kind == "topk":
        idx, val = binding.ef21_topk(state["rows"], state["k"])
        return dict(idx=idx, val=val)
    h = state["h"]
    if kind in ("grad", "csr"):
        return h.local_grad(state["x"], out=state["out"])
    if kind == "steps":
        h.set_state(x=state["x"], g_i=state["g_i"])
        for _ in range(state["steps"]):
            h.step()
        x, g_i, g = h.get_state()
        return dict(x=x, g_i=g_i, g=g)
    if kind == "update":
        h.step(state["pool"][state["at"]], state["flags"])
        state["at"] = (state["at"] + 1) % len(state["pool"])
        return h.get_x()
    gamma, L, L_i = h.theory_stepsize(state["iterations"])
    return dict(gamma=gamma, L=L, L_i=np.array(L_i))


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind, n, d = case["kind"], case["n"], case["d"]
    if kind == "topk":
        return dict(bytes=4 * n * d + 8 * n * case["k"], flops=n * d)
    if kind == "update":
        k = case["k"]
        state = 4 * n * k if case["algo"] != "ef" else 4 * n * d      # written back: k places, or every entry of e
        return dict(bytes=8 * n * d + state + 16 * d + 4 * d, flops=2 * n * d)
    if kind == "csr":
        m = case["m"]
        nnz = n * m * case["nnz"] * (0.75 if case["ragged"] else 1.0)
        return dict(bytes=8 * nnz + 8 * (n * m + 1) + 4 * n * m + 4 * n * d + 4 * d, flops=4 * nnz)
    rows = n * (case.get("tau") or case["m"])
    once = 4 * rows * d + 4 * rows
    if kind == "grad":
        return dict(bytes=once + 4 * n * d + 4 * d, flops=4 * rows * d)
    if kind == "steps":
        return dict(bytes=case["steps"] * (once + 8 * n * d + 16 * d), flops=case["steps"] * 4 * rows * d)
    # one pass over the rows serves the workers' products and the whole problem's
    return dict(bytes=case["iterations"] * once, flops=case["iterations"] * 8 * rows * d)


def tolerance(case):
    kind = case["kind"]
    if kind == "topk":
        return "exact"
    if kind == "update":
        return dict(rel=5e-7)                    # a sum of n messages per coordinate and two fused multiply-adds
    if kind == "stepsize":
        return dict(rel=1e-6)                    # norms in fp64 of products in fp32
    if kind == "steps":
        return dict(rel=1e-5)                    # gradients in fp32, several iterations
    return dict(rel=2e-6)                        # sums of m products with a d-term dot product in fp32


# ---------------------------------------------------------------- in 64 bits
def _keep_topk(v, k):
    """Positions (ascending) of the k largest magnitudes per row, ties to the lower position."""
    order = torch.sort(v.abs(), dim=1, descending=True, stable=True).indices[:, :k]
    return order.sort(dim=1).values


def _dloss(y, z, loss):
    return 2.0 * (z - y) if loss == 1 else -y * torch.sigmoid(-y * z)


def _reg_grad(x, lam):
    return 2.0 * lam * x / (1.0 + x * x).square()


def _dense_grad(A, y, x, lam, loss):
    """A [n][m][d] fp32, worker by worker."""
    out = []
    for i in range(A.shape[0]):
        Ai = A[i].double()
        r = _dloss(y[i].double(), torch.mv(Ai, x), loss)
        out.append(torch.mv(Ai.t(), r) / A.shape[1] + _reg_grad(x, lam))
    return torch.stack(out)


def _exact_steps(case, seed):
    A, y, x = _dense(case, seed)
    x = x.double()
    n, k = case["n"], case["k"]
    g_i = _dense_grad(A, y, x, LAM, 0)
    g = g_i.mean(0)
    for _ in range(case["steps"]):
        diff = _dense_grad(A, y, x, LAM, 0) - g_i
        at = _keep_topk(diff, k)
        c = torch.zeros_like(diff).scatter_(1, at, diff.gather(1, at))
        g_i = g_i + c
        g = g + c.sum(0) / n
        x = x - case["gamma"] * g
    return dict(x=x, g_i=g_i, g=g)


def _exact_csr(case, seed):
    rowptr, col, val, y, x = _csr(case, seed)
    n, m, d = case["n"], case["m"], case["d"]
    x = x.double()
    out = torch.zeros((n, d), device=DEV, dtype=torch.float64)
    for i in range(n):
        lo, hi = int(rowptr[i * m]), int(rowptr[(i + 1) * m])
        length = rowptr[i * m + 1:(i + 1) * m + 1] - rowptr[i * m:(i + 1) * m]
        row = torch.repeat_interleave(torch.arange(m, device=DEV), length)
        c, v = col[lo:hi].long(), val[lo:hi].double()
        z = torch.zeros(m, device=DEV, dtype=torch.float64).index_add_(0, row, v * x[c])
        r = _dloss(y[i].double(), z, 0) / m
        out[i].index_add_(0, c, v * r[row])
        out[i] += _reg_grad(x, LAM)
    return out


def _exact_update(case, seed):
    g0, pool = _gradients(case, seed, 1)
    s, k, n = pool[0], case["k"], case["n"]
    if case["algo"] == "ef":                     # e = 0: p = gamma s, one rounding each
        p = s * torch.tensor(np.float32(GAMMA), device=DEV)
        total = torch.zeros(case["d"], device=DEV, dtype=torch.float64)
        for i in range(n):
            at = _keep_topk(p[i:i + 1], k)[0]
            total[at] += p[i, at].double()
        return -total / n
    gamma = float(np.float32(GAMMA))
    g = g0.double().mean(0)
    rows = torch.zeros(case["d"], device=DEV, dtype=torch.float64)     # sum of the messages, or of the new rows
    for i in range(n):
        diff = s[i] - g0[i]                      # the selection is made on the rounded difference
        at = _keep_topk(diff[None], k)[0]
        if case["algo"] == "ef21":
            rows[at] += diff[at].double()
            continue
        m = g0[i].double()
        m[at] += diff[at].double()
        plain = _keep_topk(s[i:i + 1], k)[0]
        b = torch.zeros(case["d"], device=DEV, dtype=torch.float64)
        b[plain] = s[i, plain].double()
        s64 = s[i].double()
        rows += m if (m - s64).square().sum() <= (b - s64).square().sum() else b
    new_g = rows / n if case["algo"] == "plus" else g + rows / n
    return -gamma * (g if case["order"] else new_g)


def _power_start(row, d):
    """The start vector of the power iteration: entries in [0.5, 1.5) / sqrt(d) from a hash of the position."""
    h = (np.arange(d, dtype=np.uint64) * 2654435761 + 0x9e3779b9 * (row + 1)) & 0xffffffff
    h ^= h >> 15
    h = (h * 2246822519) & 0xffffffff
    h ^= h >> 13
    v = (0.5 + (h >> 8).astype(np.float64) / 16777216.0) / math.sqrt(d)
    return torch.from_numpy(v).to(DEV)


def _exact_stepsize(case, seed):
    A, _, _ = _dense(case, seed)
    n, m, d = case["n"], case["m"], case["d"]
    A = A.double()
    gram = torch.stack([A[i].t() @ A[i] / m for i in range(n)])
    every = gram.mean(0)

    def largest(M, v):
        for _ in range(case["iterations"]):
            w = M @ v
            value = float(w.norm() / v.norm())
            v = w / w.norm()
        return value

    reg = 2.0 * float(np.float32(LAM))
    L_i = np.array([0.25 * largest(gram[i], _power_start(i, d)) + reg for i in range(n)])
    L = 0.25 * largest(every, _power_start(n, d)) + reg
    alpha = case["k"] / d
    r = math.sqrt(1.0 - alpha)
    gamma = 1.0 / (L + math.sqrt(float((L_i ** 2).mean())) * ((1.0 + r) / alpha - 1.0))
    return dict(gamma=gamma, L=L, L_i=L_i)


def exact(case, seed):
    kind = case["kind"]
    if kind == "topk":
        v = _topk_rows(case, seed)
        idx = _keep_topk(v, case["k"])
        return dict(idx=idx.int(), val=v.gather(1, idx).double())
    if kind == "steps":
        return _exact_steps(case, seed)
    if kind == "csr":
        return _exact_csr(case, seed)
    if kind == "update":
        return _exact_update(case, seed)
    if kind == "stepsize":
        return _exact_stepsize(case, seed)
    A, y, x = _dense(case, seed)
    lam = 0.0 if case["loss"] == 1 else LAM
    if case["tau"]:
        rows = _batch(case, seed).long()
        A = torch.stack([A[i, rows[i]] for i in range(case["n"])])
        y = torch.stack([y[i, rows[i]] for i in range(case["n"])])
    return _dense_grad(A, y, x.double(), lam, case["loss"])
