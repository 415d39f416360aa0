"""GPU parity of the local gradients (ef21_local_grad through the C ABI) against the CPU oracle:
1e-5 relative per coordinate (fp32 kernels, fp64 oracle) plus the first-order rounding floor of the
fp32 sums (helpers.gradient_rounding_floor), which matters only where a coordinate cancels."""
import numpy as np
import pytest

from helpers import best_time, gradient_rounding_floor
from paper_2106_05203_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2106_05203_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load_library()
    return torch, binding


GUARD = 2e-5    # the median allowance of a gradient entry, as a share of the gradient's largest entry


def to_gpu(torch, a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


def assert_grads_close(got, ref, A_dense, y, x, dot_depth, sum_depth, what):
    """got, ref: [n][d]; A_dense: [n][m][d]."""
    for i in range(ref.shape[0]):
        bound = 1e-5 * np.abs(ref[i]) + gradient_rounding_floor(A_dense[i], y[i], x, dot_depth, sum_depth)
        err = np.abs(got[i].astype(np.float64) - ref[i])
        assert np.all(err <= bound), f"{what}, worker {i}: max err {err.max():.3e}, {int((err > bound).sum())} bad"
        # the floor must stay a floor: tiny next to the gradient's scale
        loose = np.median(bound) / np.max(np.abs(ref[i]))
        print(f"  {what}, worker {i}: worst coordinate uses {np.max(err / np.maximum(bound, 1e-300)):.3f} of its allowance; "
              f"median allowance {loose:.2e} of the largest entry", flush=True)
        assert loose <= GUARD, f"{what}: tolerance too loose"


def densify(W):
    D = np.zeros((W.n * W.m, W.d), np.float32)
    for r in range(W.n * W.m):
        s, e = W.rowptr[r], W.rowptr[r + 1]
        D[r, W.col[s:e]] = W.val[s:e]
    return D.reshape(W.n, W.m, W.d)


# d: vector path (d % 4 == 0) at each register tiling, scalar path, two-pass path for long rows
@pytest.mark.parametrize("n,d,m", [(4, 100, 250), (3, 256, 37), (2, 260, 64), (3, 1000, 130), (5, 2000, 301),
                                   (2, 4096, 50), (3, 99, 70), (2, 333, 41), (2, 2047, 33), (2, 4100, 29),
                                   (2, 6001, 21), (1, 1, 1)])
def test_dense_gradient(gpu, oracle, n, d, m):
    torch, binding = gpu
    print(f"dense grad case n={n} d={d} m={m}", flush=True)
    W = workloads.logreg_dense(n, d, m, seed=d + m)
    P = oracle.LogRegDense(W.A, W.y, 0.1)
    rng = np.random.default_rng(1)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, W.A), to_gpu(torch, W.y), 0.1)
        for scale in (0.0, 1.0, 8.0):
            x = (rng.standard_normal(d) * scale).astype(np.float32)
            got = h.local_grad(to_gpu(torch, x))
            again = h.local_grad(to_gpu(torch, x))
            torch.cuda.synchronize()
            ref = P.grads(x.astype(np.float64))
            assert_grads_close(got.cpu().numpy(), ref, W.A, W.y, x, d / 64 + 8, 16, f"scale {scale}")
            assert torch.equal(got, again), "the dense gradient is bitwise reproducible"
        # x = NULL uses the handle's iterate
        h.set_state(to_gpu(torch, x), None, None)
        assert torch.equal(h.local_grad(), got)


# a workgroup per row: every number of quads per thread at its ends, quads that straddle the end of the row by one,
# two and three columns, rows that are not 16-byte aligned, one row and many per block, a minibatch with an entry
# out of range; the last two take the two passes again
@pytest.mark.parametrize("n,d,m", [(1, 4100, 1), (2, 4101, 9), (2, 8192, 13), (3, 8194, 7), (2, 12288, 31), (1, 12291, 5),
                                   (2, 16384, 6), (2, 16385, 6), (1, 20481, 10), (2, 24578, 5), (300, 4097, 3),
                                   (1, 28672, 11), (1, 28673, 4), (2, 3, 5),
                                   # one block of rows per worker: more groups than between two folds of the sums,
                                   # and no second chunk where there is room for one only
                                   (300, 4100, 37), (257, 8196, 19), (257, 16388, 8)])
def test_dense_gradient_wide_rows(gpu, oracle, n, d, m):
    torch, binding = gpu
    print(f"wide dense grad case n={n} d={d} m={m}", flush=True)
    rng = np.random.default_rng(d + m)
    A = (rng.standard_normal((n, m, d), dtype=np.float32) / np.float32(np.sqrt(d)))
    y = np.where(rng.random((n, m)) < 0.5, 1.0, -1.0).astype(np.float32)
    x = rng.standard_normal(d).astype(np.float32)
    ref = oracle.LogRegDense(A, y, 0.1).grads(x.astype(np.float64))
    with binding.EF21(n, d, 1, 0.1) as h:
        pad = torch.empty(A.size + 1, device="cuda")                  # A itself at an odd 4-byte address
        Ag = pad[1:].view(n, m, d)
        Ag.copy_(torch.from_numpy(A))
        h.set_problem_dense(Ag, to_gpu(torch, y), 0.1)
        got = h.local_grad(to_gpu(torch, x))
        # additions behind one dot product: a thread's quads, six wavefront steps, sixteen wavefronts (or, in the two
        # passes, a lane's share of the row)
        depth = 4 * -(-d // 4096) + 22 if 4 <= d <= 28672 else d / 64 + 8
        if d != 28673:
            assert_grads_close(got.cpu().numpy(), ref, A, y, x, depth, 16, "wide")
        else:                                                        # as above without the check of the floor's size
            bound = 1e-5 * np.abs(ref[0]) + gradient_rounding_floor(A[0], y[0], x, depth, 16)
            assert np.all(np.abs(got.cpu().numpy()[0] - ref[0]) <= bound)
        assert torch.equal(got, h.local_grad(to_gpu(torch, x)))
        rows = torch.arange(m, dtype=torch.int32, device="cuda").repeat(n, 1).contiguous()
        h.set_minibatch(rows)
        assert torch.equal(got, h.local_grad(to_gpu(torch, x))), "all rows in order"
        if m > 1:
            batch = np.stack([rng.permutation(m) for _ in range(n)])   # another order, and another row left out, per worker
            left_out = batch[:, 0].copy()
            batch[:, 0] = m                                          # contributes nothing
            rows.copy_(torch.from_numpy(batch.astype(np.int32)))
            part = h.local_grad(to_gpu(torch, x)).cpu().numpy()
            for i in range(n):
                a, yi = A[i, left_out[i]].astype(np.float64), float(y[i, left_out[i]])
                one = -yi / (1 + np.exp(yi * (a @ x.astype(np.float64)))) * a / m
                assert np.all(np.abs(part[i] - (ref[i] - one)) <= 1e-5 * np.abs(ref).max() + 1e-6), f"worker {i}"


@pytest.mark.parametrize("n,d,m,nnz", [(3, 64, 30, 7), (4, 5000, 200, 50), (2, 50_000, 100, 500), (2, 1000, 40, 130)])
def test_csr_gradient(gpu, oracle, n, d, m, nnz):
    torch, binding = gpu
    print(f"csr grad case n={n} d={d} m={m} nnz/row={nnz}", flush=True)
    W = workloads.logreg_csr(n, d, m, nnz, seed=d + nnz)
    P = oracle.LogRegCSR(W.rowptr, W.col, W.val, W.y, n, m, d, 0.1)
    D = densify(W)
    rng = np.random.default_rng(2)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_csr(to_gpu(torch, W.rowptr, np.int64), to_gpu(torch, W.col, np.int32), to_gpu(torch, W.val),
                          to_gpu(torch, W.y), m, 0.1)
        for scale in (0.0, 1.0, 4.0):
            x = (rng.standard_normal(d) * scale).astype(np.float32)
            got = h.local_grad(to_gpu(torch, x))
            torch.cuda.synchronize()
            assert_grads_close(got.cpu().numpy(), P.grads(x.astype(np.float64)), D, W.y, x, nnz / 64 + 8, 32,
                               f"scale {scale}")


def test_csr_ragged_rows(gpu, oracle):
    """Rows of different lengths, empty rows included."""
    torch, binding = gpu
    rng = np.random.default_rng(4)
    n, m, d = 3, 50, 300
    lens = rng.integers(0, 200, size=n * m)
    lens[::9] = 0
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(d, size=L, replace=False)) for L in lens]).astype(np.int32)
    val = rng.random(col.size).astype(np.float32)
    y = np.where(rng.random((n, m)) < 0.5, 1.0, -1.0).astype(np.float32)
    P = oracle.LogRegCSR(rowptr, col, val, y, n, m, d, 0.1)
    x = rng.standard_normal(d).astype(np.float32)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_csr(to_gpu(torch, rowptr, np.int64), to_gpu(torch, col, np.int32), to_gpu(torch, val),
                          to_gpu(torch, y), m, 0.1)
        got = h.local_grad(to_gpu(torch, x))
        torch.cuda.synchronize()
    D = np.zeros((n * m, d), np.float32)
    for r in range(n * m):
        D[r, col[rowptr[r]:rowptr[r + 1]]] = val[rowptr[r]:rowptr[r + 1]]
    assert_grads_close(got.cpu().numpy(), P.grads(x.astype(np.float64)), D.reshape(n, m, d), y, x, 200 / 64 + 8, 64,
                       "ragged")


@pytest.mark.parametrize("n,m,d,always,extra", [(2, 1500, 200, (0, 5, 199), 6), (1, 17000, 70, (1,), 3),
                                                (3, 100, 13000, (12287, 12288), 40), (1, 70000, 70, (69,), 2)])
def test_csr_long_columns_many_rows(gpu, oracle, n, m, d, always, extra):
    """Columns present in every row (pieces of a column longer than a staging tile, summed by the whole
    wavefront), more rows per worker than the in-LDS coefficient vector holds, more than 16-bit row
    indices hold, columns next to a range boundary; and the sorted-CSR gradient is bitwise reproducible."""
    torch, binding = gpu
    print(f"csr long columns case n={n} m={m} d={d}", flush=True)
    rng = np.random.default_rng(m + d)
    others = np.setdiff1d(np.arange(d), np.array(always))
    rows = [np.sort(np.concatenate([np.array(always), rng.choice(others, size=extra, replace=False)]))
            for _ in range(n * m)]
    per = len(always) + extra
    rowptr = (np.arange(n * m + 1) * per).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    val = (rng.random(col.size) * 2 - 0.5).astype(np.float32)
    y = np.where(rng.random((n, m)) < 0.5, 1.0, -1.0).astype(np.float32)
    P = oracle.LogRegCSR(rowptr, col, val, y, n, m, d, 0.1)
    x = rng.standard_normal(d).astype(np.float32)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_csr(to_gpu(torch, rowptr, np.int64), to_gpu(torch, col, np.int32), to_gpu(torch, val),
                          to_gpu(torch, y), m, 0.1)
        got = h.local_grad(to_gpu(torch, x))
        again = h.local_grad(to_gpu(torch, x))
        torch.cuda.synchronize()
    assert torch.equal(got, again), "the gradient from sorted CSR rows is bitwise reproducible"
    D = np.zeros((n * m, d), np.float32)
    D[np.repeat(np.arange(n * m), per), col] = val
    assert_grads_close(got.cpu().numpy(), P.grads(x.astype(np.float64)), D.reshape(n, m, d), y, x, per / 64 + 8,
                       m / 64 + 32, "long columns")


def test_csr_unsorted_columns(gpu, oracle):
    """Columns in arbitrary order inside the rows: the library must notice and take its kernel that
    does not rely on ascending columns; same gradients."""
    torch, binding = gpu
    n, d, m, nnz = 3, 20_000, 60, 90
    W = workloads.logreg_csr(n, d, m, nnz, seed=12)
    rng = np.random.default_rng(5)
    col = W.col.reshape(n * m, nnz).copy()
    val = W.val.reshape(n * m, nnz).copy()
    for r in range(n * m):
        perm = rng.permutation(nnz)
        col[r], val[r] = col[r, perm], val[r, perm]
    P = oracle.LogRegCSR(W.rowptr, W.col, W.val, W.y, n, m, d, 0.1)
    x = rng.standard_normal(d).astype(np.float32)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_csr(to_gpu(torch, W.rowptr, np.int64), to_gpu(torch, col.reshape(-1), np.int32),
                          to_gpu(torch, val.reshape(-1)), to_gpu(torch, W.y), m, 0.1)
        got = h.local_grad(to_gpu(torch, x))
        torch.cuda.synchronize()
    assert_grads_close(got.cpu().numpy(), P.grads(x.astype(np.float64)), densify(W), W.y, x, nnz / 64 + 8, 64,
                       "unsorted")


@pytest.mark.timeout(400)
def test_config2_full_size_gradient(gpu, oracle):
    """Config 2 at full size (n = 20, m = 5000, d = 2000, 800 MB of rows): every worker's gradient, at
    x = 0 (closed form -A^T y / 2m inside the oracle's pins) and at a random x."""
    torch, binding = gpu
    c = workloads.CONFIGS["C2"]
    n, d, m = c["n"], c["d"], c["m"]
    print("C2 full size gradient", flush=True)
    W = workloads.logreg_dense(n, d, m, seed=c["seed"])
    P = oracle.LogRegDense(W.A, W.y, c["lam"])
    rng = np.random.default_rng(21)
    with binding.EF21(n, d, c["k"], c["gamma"]) as h:
        h.set_problem_dense(to_gpu(torch, W.A), to_gpu(torch, W.y), c["lam"])
        for x in (np.zeros(d, np.float32), rng.standard_normal(d).astype(np.float32)):
            got = h.local_grad(to_gpu(torch, x))
            again = h.local_grad(to_gpu(torch, x))
            torch.cuda.synchronize()
            assert torch.equal(got, again)
            assert_grads_close(got.cpu().numpy(), P.grads(x.astype(np.float64)), W.A, W.y, x, d / 64 + 8, 16,
                               "C2 full size")


@pytest.mark.timeout(600)
def test_config3_full_size_gradient(gpu, oracle):
    """Config 3 at full size (n = 100, m = 2000, d = 50000, 10^8 non-zeros): three workers' gradients
    coordinate by coordinate (the rounding floor needs the worker's matrix), all workers through the
    norm of the difference."""
    import scipy.sparse as sp
    torch, binding = gpu
    c = workloads.CONFIGS["C3"]
    n, d, m, nnz = c["n"], c["d"], c["m"], c["nnz_per_row"]
    print("C3 full size gradient", flush=True)
    W = workloads.logreg_csr(n, d, m, nnz, seed=c["seed"])
    P = oracle.LogRegCSR(W.rowptr, W.col, W.val, W.y, n, m, d, c["lam"])
    rng = np.random.default_rng(22)
    x = rng.standard_normal(d).astype(np.float32)
    with binding.EF21(n, d, c["k"], c["gamma"]) as h:
        h.set_problem_csr(to_gpu(torch, W.rowptr, np.int64), to_gpu(torch, W.col, np.int32), to_gpu(torch, W.val),
                          to_gpu(torch, W.y), m, c["lam"])
        got = h.local_grad(to_gpu(torch, x))
        again = h.local_grad(to_gpu(torch, x))
        torch.cuda.synchronize()
        assert torch.equal(got, again)
    got = got.cpu().numpy()
    ref = P.grads(x.astype(np.float64))
    for i in (0, 57, 99):
        lo, hi = W.rowptr[i * m], W.rowptr[(i + 1) * m]
        A_i = sp.csr_matrix((W.val[lo:hi], W.col[lo:hi], W.rowptr[i * m:(i + 1) * m + 1] - lo), shape=(m, d))
        bound = 1e-5 * np.abs(ref[i]) + gradient_rounding_floor(A_i, W.y[i], x, nnz / 64 + 8, 64)
        err = np.abs(got[i].astype(np.float64) - ref[i])
        assert np.all(err <= bound), f"worker {i}: max err {err.max():.3e}, {int((err > bound).sum())} bad"
        assert np.median(bound) <= 2e-5 * np.max(np.abs(ref[i]))
    rel = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert rel.max() <= 1e-6, f"relative error of the gradients in the 2-norm: {rel.max():.3e}"


# groups of 16, 32 and 64 lanes per row at their ends, rows of 1 to 5 columns, with 32 entries per lane in flight and
# (problems of more than 2^24 entries) with 64; A at an odd 4-byte address, a minibatch with an entry out of range
@pytest.mark.parametrize("n,d,m", [(2, 1, 9), (3, 2, 70), (2, 3, 33), (2, 4, 65), (3, 5, 40), (2, 63, 129), (2, 64, 31),
                                   (3, 65, 64), (2, 127, 200), (2, 129, 17), (2, 257, 90), (40, 515, 30), (2, 1023, 70),
                                   (1, 1026, 19), (2, 2048, 12), (2, 61, 140_000), (2, 126, 70_000), (2, 251, 34_000),
                                   (2, 509, 17_000), (2, 1021, 8_500)])
def test_dense_gradient_short_rows(gpu, oracle, n, d, m):
    torch, binding = gpu
    print(f"short dense grad case n={n} d={d} m={m}", flush=True)
    rng = np.random.default_rng(d + m)
    A = rng.standard_normal((n, m, d), dtype=np.float32) / np.float32(np.sqrt(d))
    y = np.where(rng.random((n, m)) < 0.5, 1.0, -1.0).astype(np.float32)
    x = rng.standard_normal(d).astype(np.float32)
    x64 = x.astype(np.float64)

    def grads_of(rows, tau):
        """rows: the row numbers of each worker; the sums are divided by tau."""
        out = []
        for i in range(n):
            Ai = A[i, rows[i]].astype(np.float64)
            r = -y[i, rows[i]] / (1.0 + np.exp(y[i, rows[i]] * (Ai @ x64)))
            out.append(Ai.T @ r / tau + 0.2 * x64 / (1.0 + x64 * x64) ** 2)
        return np.stack(out)

    with binding.EF21(n, d, 1, 0.1) as h:
        pad = torch.empty(A.size + 1, device="cuda")
        Ag = pad[1:].view(n, m, d)
        Ag.copy_(torch.from_numpy(A))
        h.set_problem_dense(Ag, to_gpu(torch, y), 0.1)
        got = h.local_grad(to_gpu(torch, x))
        assert torch.equal(got, h.local_grad(to_gpu(torch, x)))
        ref = grads_of([np.arange(m)] * n, m)
        # additions behind a sum over rows: a group's trips and the two to eight levels that join the blocks
        depth = d / 64 + 8
        for i in range(n):
            bound = 1e-5 * np.abs(ref[i]) + gradient_rounding_floor(A[i], y[i], x, depth, 16)
            assert np.all(np.abs(got.cpu().numpy()[i] - ref[i]) <= bound)
        if d <= 8192 and m < 10_000:                           # the same sums finished by the Top-k kernel
            h.set_state(x=to_gpu(torch, x), g_i=torch.zeros((n, d), device="cuda"))
            h.step()
            idx, val = h.get_messages()
            assert torch.equal(val, got.gather(1, idx.long()))
        tau = max(1, m // 3)
        batch = np.stack([rng.permutation(m)[:tau] for _ in range(n)]).astype(np.int32)
        out_of_range = (np.arange(n), rng.integers(tau, size=n))          # one place per worker
        for wrong in (None, -1, m, 2 ** 31 - 1):
            rows = [batch[i] for i in range(n)]
            if wrong is not None:
                given = batch.copy()
                given[out_of_range] = wrong
                rows = [np.delete(batch[i], out_of_range[1][i]) for i in range(n)]
            h.set_minibatch(to_gpu(torch, batch if wrong is None else given, np.int32))
            ref = grads_of(rows, tau)
            got = h.local_grad(to_gpu(torch, x)).cpu().numpy()
            for i in range(n):
                bound = 1e-5 * np.abs(ref[i]) + gradient_rounding_floor(A[i][batch[i]], y[i][batch[i]], x, depth, 16)
                assert np.all(np.abs(got[i] - ref[i]) <= bound), f"worker {i}, entry {wrong}"


# one segment group per wavefront and four (192 workgroups and more), rows and columns past the last group
@pytest.mark.parametrize("n,d,m,nnz", [(191, 70, 66, 3), (192, 70, 66, 3), (192, 2049, 65, 4), (2, 600, 2050, 7)])
def test_csr_gradient_groups(gpu, oracle, n, d, m, nnz):
    torch, binding = gpu
    print(f"csr groups case n={n} d={d} m={m} nnz/row={nnz}", flush=True)
    W = workloads.logreg_csr(n, d, m, nnz, seed=d + n)
    x = np.random.default_rng(5).standard_normal(d).astype(np.float32)
    P = oracle.LogRegCSR(W.rowptr, W.col, W.val, W.y, n, m, d, 0.1)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_csr(to_gpu(torch, W.rowptr, np.int64), to_gpu(torch, W.col, np.int32), to_gpu(torch, W.val),
                          to_gpu(torch, W.y), m, 0.1)
        got = h.local_grad(to_gpu(torch, x))
        assert_grads_close(got.cpu().numpy(), P.grads(x.astype(np.float64)), densify(W), W.y, x, nnz / 64 + 8, 32, "groups")


# an infinity in a row that a group of rows only carries along: worker 0's first row (loaded by every worker of the
# workgroup-per-row kernel in place of rows it does not have), a worker's last row (in place of rows past the block), and
# row 0 outside the minibatch beside an entry out of range
@pytest.mark.parametrize("n,d,m", [(3, 4097, 7), (2, 8192, 9), (3, 9000, 15), (2, 16384, 63), (2, 20001, 5), (3, 1, 9),
                                   (3, 4, 33), (2, 60, 37), (2, 61, 70), (2, 120, 41), (3, 200, 19), (2, 500, 13),
                                   (2, 1000, 11), (2, 2000, 21), (2, 2047, 21), (2, 3000, 9), (2, 29000, 5),
                                   (2, 60, 150_000)])
def test_an_infinite_entry_stays_in_its_row(gpu, n, d, m):
    torch, binding = gpu
    print(f"infinite entry case n={n} d={d} m={m}", flush=True)
    rng = np.random.default_rng(d + m)
    A = rng.standard_normal((n, m, d), dtype=np.float32) / np.float32(np.sqrt(d))
    y = np.ones((n, m), np.float32)
    x = -np.abs(rng.standard_normal(d)).astype(np.float32) - np.float32(0.1)    # every product with +inf is -inf
    x64 = x.astype(np.float64)
    A[0, 0, rng.integers(min(4, d))] = np.inf         # z = -inf: the coefficient is -1, the gradient's entry -inf
    A[n - 1, m - 1, rng.integers(d)] = np.inf

    def grads_of(rows, tau):
        """rows [n][..]: valid row numbers; the sum is divided by tau."""
        out = np.empty((n, d))
        for i in range(n):
            Ai, yi = A[i, rows[i]].astype(np.float64), y[i, rows[i]].astype(np.float64)
            with np.errstate(over="ignore"):
                r = -yi / (1.0 + np.exp(yi * (Ai @ x64)))
            out[i] = r @ Ai / tau + 0.2 * x64 / (1.0 + x64 * x64) ** 2
        return out

    def check(got, ref, what):
        assert np.array_equal(np.isfinite(got), np.isfinite(ref)), f"{what}: {np.argwhere(np.isfinite(got) != np.isfinite(ref))[:4]}"
        fin = np.isfinite(ref)
        assert np.array_equal(got[~fin], ref[~fin]), what
        assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-4 * np.abs(ref[fin]).max()), what    # the values: the tests above

    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.1)
        check(h.local_grad(to_gpu(torch, x)).cpu().numpy(), grads_of([np.arange(m)] * n, m), "all rows")
        if m > 2:
            batch = np.stack([1 + rng.permutation(m - 2) for _ in range(n)]).astype(np.int32)   # neither infinite row
            tau = batch.shape[1]
            h.set_minibatch(to_gpu(torch, batch, np.int32))
            check(h.local_grad(to_gpu(torch, x)).cpu().numpy(), grads_of(batch, tau), "batch")
            batch[:, tau // 2] = m
            h.set_minibatch(to_gpu(torch, batch, np.int32))
            check(h.local_grad(to_gpu(torch, x)).cpu().numpy(), grads_of(np.delete(batch, tau // 2, axis=1), tau), "entry out of range")


# step finishes the gradient's sums in the Top-k kernel or before it, by their number and the row's length: the same bits
# as local_grad on both sides, and not one workgroup per worker where there are many (long rows, few workers)
@pytest.mark.parametrize("n,d,m", [(1, 8000, 1000), (2, 8192, 500), (1, 4097, 3000), (2, 4096, 60), (32, 8000, 9),
                                   (2, 2000, 2000), (4, 1000, 2000), (10, 2000, 40), (2, 300, 5000)])
def test_step_finishes_the_gradient_either_way(gpu, n, d, m):
    torch, binding = gpu
    print(f"finish case n={n} d={d} m={m}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(d + m)
    A = torch.randn((n, m, d), device="cuda", generator=g) / d ** 0.5
    y = torch.where(torch.rand((n, m), device="cuda", generator=g) < 0.5, 1.0, -1.0)
    x = torch.randn(d, device="cuda", generator=g)
    with binding.EF21(n, d, 5, 1e-30) as h:
        h.set_problem_dense(A, y, 0.1)
        want = h.local_grad(x)
        h.set_state(x=x, g_i=torch.zeros((n, d), device="cuda"))
        h.step()
        idx, val = h.get_messages()
        assert torch.equal(val, want.gather(1, idx.long()))
        kept = val.abs().min(1).values
        rest = want.scatter(1, idx.long(), 0.0).abs().max(1).values
        assert (rest <= kept).all()
        out = torch.empty((n, d), device="cuda")
        grad, step = best_time(torch, lambda: h.local_grad(x, out=out)), best_time(torch, h.step)
    print(f"  local_grad {grad:.0f} us, step {step:.0f} us", flush=True)
    assert step <= grad + 35.0, (grad, step)


# the same rows with one or two workers and with sixteen: few workers fill the chip by cutting their rows into more blocks
@pytest.mark.parametrize("n,d,m", [(1, 80, 100_000), (2, 100, 40_000), (1, 1000, 8000)])
def test_few_workers_fill_the_chip(gpu, n, d, m):
    torch, binding = gpu
    print(f"few workers case n={n} d={d} m={m}", flush=True)
    times = {}
    for workers in (n, 16):
        rows = n * m // workers
        A = torch.randn((workers, rows, d), device="cuda")
        y = torch.ones((workers, rows), device="cuda")
        x = torch.zeros(d, device="cuda")
        out = torch.empty((workers, d), device="cuda")
        with binding.EF21(workers, d, 1, 0.1) as h:
            h.set_problem_dense(A, y, 0.1)
            h.local_grad(x, out=out)
            # at x = 0 every coefficient is -1/2: the gradient is the rows' mean times that
            want = -0.5 * A.double().mean(1)
            assert (out.double() - want).abs().max() <= 1e-5 * want.abs().max() + 1e-7
            times[workers] = best_time(torch, lambda: h.local_grad(x, out=out))
    print(f"  {times}", flush=True)
    assert times[n] <= 2.0 * times[16] + 10.0, times


# the kernels that add a column's partial sums: a thread per column (up to 16 blocks, or many columns), eight threads with up to
# 8 and up to 16 entries of a chain in flight, each with a last, partial group of 64 columns, and the sums left to the Top-k kernel: an
# iteration from the reported gradient and one that forms its own agree bit for bit (both add the chains in the same order)
@pytest.mark.parametrize("n,d,m", [(2, 100, 700), (30, 70, 1600), (3, 130, 5000), (1, 65, 9000), (1, 1, 20000), (2, 300, 60000),
                                   (1, 1001, 3000), (12, 3000, 400), (8, 5000, 300), (3, 900, 640), (3, 901, 640), (14, 600, 4000), (1, 224, 40000)])
def test_partial_sums_of_many_blocks(gpu, n, d, m, kept=None):
    torch, binding = gpu
    print(f"partial sums n={n} d={d} m={m}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(d + m)
    A = torch.randn((n, m, d), device="cuda", generator=g) / d ** 0.5
    y = torch.where(torch.rand((n, m), device="cuda", generator=g) < 0.5, 1.0, -1.0)
    x = 0.3 * torch.randn(d, device="cuda", generator=g)
    k = kept or max(1, d // 20)
    with binding.EF21(n, d, k, 0.3) as own, binding.EF21(n, d, k, 0.3) as given:
        for h in (own, given):
            h.set_problem_dense(A, y, 0.1)
            h.set_state(x, torch.zeros((n, d), device="cuda"), None)
        s = given.local_grad()
        # fp64 on the GPU; per entry the first-order rounding of helpers.gradient_rounding_floor: margins summed in d / 64 + 8
        # levels with curvature 1/4, sums of a block's rows in fp32, 16 levels and a chain of up to 64 rows per lane
        z = torch.stack([torch.mv(A[i].double(), x.double()) for i in range(n)])
        coef = -y * torch.sigmoid(-y.double() * z)
        ref = torch.stack([torch.mv(A[i].double().t(), coef[i]) / m for i in range(n)]) + 0.2 * x.double() / (1 + x.double() ** 2) ** 2
        u = 2.0 ** -24
        dz = torch.stack([(d / 64 + 8) * u * torch.mv(A[i].abs().double(), x.abs().double()) for i in range(n)])
        dcoef = 0.25 * dz + 32 * u * coef.abs()
        bound = 1e-6 * ref.abs() + torch.stack([torch.mv(A[i].abs().double().t(), dcoef[i]) / m for i in range(n)]) + u
        assert bool(((s.double() - ref).abs() <= bound).all())
        for _ in range(3):
            own.step()
            given.step(given.local_grad())
            for a, b in zip(own.get_state(), given.get_state()):
                assert torch.equal(a, b)
            for a, b in zip(own.get_messages(), given.get_messages()):
                assert torch.equal(a, b)


# few rows: up to four sums per column are left to the Top-k kernel up to 1200 columns, and up to 4096 where more than an eighth of
# the row (or more than 1024 entries) is kept
@pytest.mark.parametrize("n,d,m,k", [(3, 901, 8, 40), (3, 1200, 32, 150), (3, 1201, 32, 150), (3, 1200, 33, 150), (2, 1200, 3, 151),
                                     (2, 4096, 32, 513), (2, 4096, 7, 1025), (2, 4097, 7, 1025), (1, 4096, 40, 2000)])
def test_few_sums_left_to_the_selection(gpu, n, d, m, k):
    test_partial_sums_of_many_blocks(gpu, n, d, m, k)
