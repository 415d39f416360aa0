"""GPU parity of ef21_theory_stepsize against the oracle's exact eigenvalues: the power iteration approaches
every smoothness constant from below, to 1e-4 where the matrix has a dominant direction and to two per cent
on matrices without one (the gap of a random matrix's top eigenvalues is small), and the stepsize follows."""
import time

import numpy as np
import pytest

from paper_2106_05203_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2106_05203_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load_library()
    return torch, binding


def to_gpu(torch, a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


def check(got, exact, below, what):
    got, exact = np.asarray(got), np.asarray(exact)
    assert np.all(got <= exact * (1 + 2e-6)), f"{what}: an estimate above the eigenvalue: {got} vs {exact}"
    assert np.all(got >= exact * (1 - below)), f"{what}: {got} vs {exact}"


@pytest.mark.parametrize("n,d,m,k", [(4, 100, 250, 3), (3, 333, 41, 10), (2, 4100, 29, 41)])
@pytest.mark.parametrize("loss", ["logistic", "squares"])
def test_dense_with_a_dominant_direction(gpu, oracle, n, d, m, k, loss):
    """Rows with a common offset (non-negative features, as in the paper's data sets) have one large eigenvalue."""
    torch, binding = gpu
    print(f"stepsize dense n={n} d={d} m={m} {loss}", flush=True)
    rng = np.random.default_rng(d)
    A = (rng.standard_normal((n, m, d)) / np.sqrt(d) + 0.5 * rng.random((n, 1, d)) / np.sqrt(d)).astype(np.float32)
    A *= np.linspace(0.5, 2.0, n)[:, None, None].astype(np.float32)          # workers of different scale
    t = np.where(rng.random((n, m)) < 0.5, 1.0, -1.0).astype(np.float32)
    lam = 0.1
    P = oracle.LeastSquaresDense(A, t, lam) if loss == "squares" else oracle.LogRegDense(A, t, lam)
    L_i = oracle.smoothness_constants(P)
    with binding.EF21(n, d, k, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, t), lam)
        if loss == "squares":
            h.set_loss(binding.LOSS_LEAST_SQUARES)
        gamma, L, got_i = h.theory_stepsize(150)
    check(got_i, L_i, 1e-4, "L_i")
    L_exact = oracle.smoothness_constant_of_f(P)
    check([L], [L_exact], 1e-4, "L")
    ref = oracle.theory_stepsize(L_i, k / d, L=L_exact)
    assert ref * (1 - 2e-6) <= gamma <= ref * (1 + 2e-4)
    assert L <= np.mean(got_i) * (1 + 1e-6)                      # the remark before Theorem 1: L <= mean L_i


def test_dense_without_a_dominant_direction(gpu, oracle):
    torch, binding = gpu
    n, d, m, k = 3, 200, 500, 2
    W = workloads.logreg_dense(n, d, m, seed=3)
    P = oracle.LogRegDense(W.A, W.y, 0.1)
    L_i = oracle.smoothness_constants(P)
    with binding.EF21(n, d, k, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, W.A), to_gpu(torch, W.y), 0.1)
        few = h.theory_stepsize(5)
        many = h.theory_stepsize(300)
    check(many[2], L_i, 2e-2, "L_i after 300 steps")
    check(few[2], L_i, 0.6, "L_i after 5 steps")
    assert np.all(np.asarray(few[2]) <= np.asarray(many[2]) * (1 + 1e-6))     # the estimate grows with the steps
    ref = oracle.theory_stepsize(L_i, k / d, L=oracle.smoothness_constant_of_f(P))
    assert ref * (1 - 2e-6) <= many[0] <= ref * 1.03


@pytest.mark.parametrize("sorted_cols", [True, False])
def test_csr(gpu, oracle, sorted_cols):
    torch, binding = gpu
    n, d, m, nnz, k = 3, 3000, 150, 40, 30
    W = workloads.logreg_csr(n, d, m, nnz, seed=4)
    col, val = np.array(W.col), np.abs(np.array(W.val))           # non-negative features: a dominant direction
    if not sorted_cols:
        for r in range(n * m):
            s, e = W.rowptr[r], W.rowptr[r + 1]
            col[s:e], val[s:e] = col[s:e][::-1].copy(), val[s:e][::-1].copy()
    P = oracle.LogRegCSR(W.rowptr, col, val, W.y, n, m, d, 0.05)
    L_i = oracle.smoothness_constants(P)
    with binding.EF21(n, d, k, 0.1) as h:
        h.set_problem_csr(to_gpu(torch, W.rowptr, np.int64), to_gpu(torch, col, np.int32), to_gpu(torch, val),
                          to_gpu(torch, W.y), m, 0.05)
        gamma, L, got_i = h.theory_stepsize(200)
    check(got_i, L_i, 1e-3, "L_i")
    L_exact = oracle.smoothness_constant_of_f(P)
    check([L], [L_exact], 1e-3, "L")
    ref = oracle.theory_stepsize(L_i, k / d, L=L_exact)
    assert ref * (1 - 2e-6) <= gamma <= ref * (1 + 2e-3)


def test_stepsize_runs_ef21_downhill(gpu, oracle):
    """EF21 with the stepsize the library computes: f decreases along the run, as Theorem 1's proof shows for the
    Lyapunov function; here checked on f at the end against the start."""
    torch, binding = gpu
    n, d, m, k = 4, 100, 250, 2
    W = workloads.logreg_dense(n, d, m, seed=5)
    P = oracle.LogRegDense(W.A, W.y, 0.1)
    with binding.EF21(n, d, k, 0.1) as probe:
        probe.set_problem_dense(to_gpu(torch, W.A), to_gpu(torch, W.y), 0.1)
        gamma = probe.theory_stepsize(300)[0]
    x0 = np.random.default_rng(6).standard_normal(d).astype(np.float32)
    with binding.EF21(n, d, k, gamma) as h:
        h.set_problem_dense(to_gpu(torch, W.A), to_gpu(torch, W.y), 0.1)
        x0g = to_gpu(torch, x0)
        h.set_state(x0g, h.local_grad(x0g), None)
        for _ in range(200):
            h.step()
        assert P.loss(h.get_x().cpu().numpy().astype(np.float64)) < P.loss(x0.astype(np.float64))


def test_argument_errors(gpu):
    torch, binding = gpu
    with binding.EF21(2, 16, 2, 0.1) as h:
        with pytest.raises(binding.EF21Error):
            h.theory_stepsize(10)                                 # no problem
        A = torch.ones((2, 5, 16), device="cuda")
        h.set_problem_dense(A, torch.ones((2, 5), device="cuda"), 0.0)
        with pytest.raises(binding.EF21Error):
            h.theory_stepsize(0)
        gamma, L, L_i = h.theory_stepsize(3)                      # rank one: lambda_max = |a|^2 = 16 exactly
        assert L_i == pytest.approx([4.0, 4.0], rel=1e-6) and L == pytest.approx(4.0, rel=1e-6)


def power_values(A, steps):
    """|w| / |v| after `steps` steps of the power iteration per worker and for the whole problem, in fp64 from the
    library's start vectors (fp32 values)."""
    n, m, d = A.shape
    A = A.astype(np.float64)
    G = [a.T @ a / m for a in A]
    G.append(sum(G) / n)
    out = []
    for row, g in enumerate(G):
        h = (np.arange(d, dtype=np.uint64) * 2654435761 + 0x9e3779b9 * (row + 1)) & 0xffffffff
        h ^= h >> 15
        h = (h * 2246822519) & 0xffffffff
        h ^= h >> 13
        v = (0.5 + (h >> 8).astype(np.float64) / 16777216.0) / np.sqrt(d)
        for _ in range(steps):
            w = g @ v
            value = np.linalg.norm(w) / np.linalg.norm(v)
            v = w / value if value > 0 else v
        out.append(value)
    return np.array(out)


# the iteration on Gram matrices (one launch, up to 320 columns; a launch per step, up to 1024; products with a power) at the
# ends of its tiles, one row, ragged chunks of rows, several chunks, and the first size past them.  Which way a call goes
# is gram_way's matter (csrc/gram_way.h): REACHED below has shapes for each of them, which tests/test_stepsize_ways.py holds to it
@pytest.mark.parametrize("n,d,m", [(1, 1, 1), (2, 31, 7), (3, 32, 300), (1, 33, 1), (2, 64, 1025), (2, 65, 515),
                                   (2, 129, 33), (5, 192, 64), (2, 193, 2), (3, 256, 770), (2, 257, 9), (2, 319, 40),
                                   (3, 320, 64), (2, 321, 31), (2, 352, 700), (1, 1023, 17), (2, 1024, 260), (1, 1025, 16)])
def test_power_iteration_value(gpu, n, d, m):
    """Non-negative features: every entry of the Gram matrix is a sum of positive terms, so rounding it to fp32 moves
    |G v| by at most 2^-24 of itself; the start vector and the product with A (1025 columns) add roundings of that
    size, which the iteration averages: 1e-6 after one to forty steps."""
    torch, binding = gpu
    print(f"power iteration n={n} d={d} m={m}", flush=True)
    rng = np.random.default_rng(d * 7 + m)
    A = rng.random((n, m, d)).astype(np.float32) * np.linspace(0.5, 2.0, n)[:, None, None].astype(np.float32)
    t = np.zeros((n, m), dtype=np.float32)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, t), 0.0)
        for steps in (40, 7, 1):
            _, L, L_i = h.theory_stepsize(steps)
            got = 4.0 * np.array(list(L_i) + [L])
            np.testing.assert_allclose(got, power_values(A, steps), rtol=1e-6, err_msg=f"{steps} steps")
        h.set_problem_dense(to_gpu(torch, 3.0 * A), to_gpu(torch, t), 0.0)     # new data behind the same handle
        _, L, L_i = h.theory_stepsize(40)
        np.testing.assert_allclose(4.0 * np.array(list(L_i) + [L]), power_values(3.0 * A, 40), rtol=1e-6)
        h.set_problem_dense(to_gpu(torch, 0.0 * A), to_gpu(torch, t), 0.0)
        _, L, L_i = h.theory_stepsize(40)
        assert L == 0.0 and not np.any(L_i)


# more iterations than one launch of the resident kernel runs (4096): it goes on from the vectors the launch before left (up to 128
# columns; 300 are squared, and see REACHED).  Two close eigenvalues, so that the last thousand iterations still move the value
@pytest.mark.parametrize("d", [40, 300])
def test_power_iteration_goes_on_over_launches(gpu, d):
    torch, binding = gpu
    n, m = 2, d
    A = np.zeros((n, m, d), np.float32)
    for i in range(n):                                    # A_i^T A_i / m diagonal, eigenvalues 1, 0.9998, and small ones
        scale = np.full(d, 0.05, np.float32)
        scale[1 + i], scale[7 + i] = 1.0, 0.9999
        A[i][np.arange(d), np.arange(d)] = np.sqrt(np.float32(m)) * scale
    y = np.zeros((n, m), np.float32)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.0)
        for steps in (4096, 4097, 5000, 8300):
            _, L, L_i = h.theory_stepsize(steps)
            got = 4.0 * np.array(list(L_i) + [L])
            want = power_values(A, steps)
            # fp32 entries of G, fp64 everywhere else: as in test_power_iteration_value
            np.testing.assert_allclose(got, want, rtol=1e-6, err_msg=f"{steps} steps")


# the first and last numbers of iterations that run as a Lanczos recurrence and those beside them (47, 2823: the power
# iteration), one row and four rows of the tridiagonal matrix per lane (177 and 178 iterations: 65 and 66 steps).  Of two workers' matrices
# this is so up to 128 columns; more columns are squared for most of these numbers, see REACHED for the recurrence's other forms
@pytest.mark.parametrize("d", [2, 64, 65, 192, 256, 320, 321, 700])
def test_recurrence_gives_the_power_iterations_value(gpu, d):
    torch, binding = gpu
    print(f"recurrence d={d}", flush=True)
    n, m = 2, d
    rng = np.random.default_rng(d)
    A = np.zeros((n, m, d), np.float32)                   # A_i^T A_i / m diagonal: one product per entry, exact in fp64
    for i in range(n):
        scale = rng.random(d).astype(np.float32)          # many eigenvalues, the largest ones close to one another
        scale[0], scale[d - 1] = 1.0, 0.9995
        A[i][np.arange(d), np.arange(d)] = np.sqrt(np.float32(m)) * scale * np.float32(1 + i)
    y = np.zeros((n, m), np.float32)
    diagonals = np.array([np.diagonal(a).astype(np.float64) ** 2 / m for a in A])
    rounded = np.vstack([diagonals, diagonals.mean(0)]).astype(np.float32).astype(np.float64)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.0)
        for steps in (47, 48, 100, 177, 178, 2822, 2823):
            _, L, L_i = h.theory_stepsize(steps)
            got = 4.0 * np.array(list(L_i) + [L])
            # fp64 on both sides from the same fp32 matrix.  The start vectors' fp32 entries may differ by a rounding (the
            # device's 1 / sqrt(d)), 2^-23: each weight in the two moments by 2^-22, and the estimate by half that times
            # the spread of the eigenvalues that still count, those above 0.9 (0.9^94 = 5e-5): 2^-23 * 0.2 = 2.4e-8.
            # Half the steps would be 1e-5 off.
            np.testing.assert_allclose(got, diagonal_power(rounded, steps), rtol=2.4e-8, err_msg=f"{steps} iterations")


def matrices_of_a_kind(kind, n, m, d, rng):
    A = rng.standard_normal((n, m, d))
    if kind == "non-negative":                            # one dominant eigenvalue
        A = rng.random((n, m, d))
    if kind == "rank 3":                                  # the recurrence ends after three steps, in exact arithmetic
        A = rng.standard_normal((n, m, 3)) @ rng.standard_normal((n, 3, d))
    if kind == "badly scaled":                            # eigenvalues over twelve orders of magnitude
        A = A * 10.0 ** -np.linspace(0, 6, d)
    if kind == "one entry":                               # rank one, in a direction the start vector hardly has
        A = np.zeros((n, m, d))
        A[:, 0, d // 2] = 3.0
    if kind == "zero":
        A = np.zeros((n, m, d))
    return A.astype(np.float32)


@pytest.mark.parametrize("kind", ["Gaussian", "non-negative", "rank 3", "badly scaled", "one entry", "zero"])
@pytest.mark.parametrize("d", [5, 40, 300, 320, 700])         # fewer columns than steps; from 300 on by squaring
def test_recurrence_on_kinds_of_matrices(gpu, kind, d):
    torch, binding = gpu
    print(f"recurrence on {kind} matrices, d={d}", flush=True)
    n, m, lam = 2, 500, 0.0 if kind != "zero" else 0.125
    A = matrices_of_a_kind(kind, n, m, d, np.random.default_rng(d))
    G = np.array([a.astype(np.float64).T @ a.astype(np.float64) / m for a in A])
    G = np.concatenate([G, G.mean(0)[None]]).astype(np.float32).astype(np.float64)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, np.zeros((n, m), np.float32)), lam)
        for steps in (48, 100, 400, 2822):
            _, L, L_i = h.theory_stepsize(steps)
            got = 4.0 * (np.array(list(L_i) + [L]) - 2.0 * lam)
            want = np.array([power_estimate(G[row], row, steps) for row in range(n + 1)])
            # The start vectors' entries may differ by 2^-23 (see above): each weight in the two moments by 2^-22, the estimate by
            # at most half of that.  The matrices are rounded to fp32 on both sides from sums in fp64 that differ in their
            # last bits: an entry may fall to the other side, 2^-24 of it, a vanishing part of the whole.
            np.testing.assert_allclose(got, want, rtol=2.0 ** -23, err_msg=f"{steps} iterations")


def power_estimate(G, row, steps):
    v = start_vector(G.shape[0], row)
    for _ in range(steps - 1):
        v = G @ v
        size = np.linalg.norm(v)
        if size == 0.0:
            return 0.0
        v /= size
    return np.linalg.norm(G @ v) / np.linalg.norm(v)


def start_vector(d, row):
    h = (np.arange(d, dtype=np.uint64) * 2654435761 + 0x9e3779b9 * (row + 1)) & 0xffffffff
    h ^= h >> 15
    h = (h * 2246822519) & 0xffffffff
    h ^= h >> 13
    return ((0.5 + (h >> 8).astype(np.float32) * np.float32(1 / 16777216)) / np.sqrt(np.float32(d))).astype(np.float64)


def diagonal_power(eigenvalues, steps):
    out = []
    for row, e in enumerate(eigenvalues):
        v = start_vector(e.size, row)
        for _ in range(steps - 1):
            v = e * v
            v /= np.linalg.norm(v)
        out.append(np.linalg.norm(e * v) / np.linalg.norm(v))
    return np.array(out)


def test_few_iterations_on_large_matrices(gpu):
    """32 workers, 1000 columns: forming 33 matrices of a million entries takes as long as a dozen iterations with the
    468 rows per worker, and an iteration on them 32 us against 40, so twenty iterations run with A: 3.4 times as long as
    five, where forming the matrices made it 4.5."""
    torch, binding = gpu
    n, d, m = 32, 1000, 468
    A = torch.randn((n, m, d), device="cuda") / d ** 0.5
    y = torch.ones((n, m), device="cuda")
    times = {}
    with binding.EF21(n, d, 10, 0.1) as h:
        h.set_problem_dense(A, y, 0.1)
        for iterations in (5, 20):
            h.theory_stepsize(iterations)
            best = np.inf
            for _ in range(5):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                h.theory_stepsize(iterations)
                best = min(best, time.perf_counter() - t0)
            times[iterations] = 1e6 * best
    print(times, flush=True)
    assert times[20] <= 3.9 * times[5], times


# powers by squaring (more than 128 columns): the ends of the groups of sixteen columns and of the strips of four groups, one row of A and
# several chunks (whether the exponent is right these matrices cannot show: REACHED)
@pytest.mark.parametrize("n,d,m", [(1, 129, 40), (3, 143, 1), (2, 145, 600), (4, 176, 33), (2, 209, 80), (2, 305, 64), (2, 320, 30),
                                   (3, 337, 50), (2, 500, 17), (1, 1009, 40), (2, 1024, 12)])
def test_powers_by_squaring_give_the_power_iterations_value(gpu, n, d, m):
    """Against the power iteration in fp64.  Non-negative features: 1e-6, as in test_power_iteration_value.  One worker's rows are zero, one's
    of the order of 1e-12, the first one's of 1e12 (the mean over the workers then is the first one's share to fp32)."""
    torch, binding = gpu
    print(f"squaring n={n} d={d} m={m}", flush=True)
    rng = np.random.default_rng(d + m)
    scale = np.array([1e12, 1e-12, 0.0, 1.0][:n], np.float32)
    A = rng.random((n, m, d)).astype(np.float32) * scale[:, None, None]
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(to_gpu(torch, A), torch.zeros((n, m), device="cuda"), 0.0)
        for steps in (2, 65, 48, 100, 128, 1001, 100000, 64):
            _, L, L_i = h.theory_stepsize(steps)
            got = 4.0 * np.array(list(L_i) + [L])
            # the product with a rank-one dominated matrix settles within a few steps: 200 stand for more
            np.testing.assert_allclose(got, power_values(A, min(steps, 200)), rtol=1e-6, err_msg=f"{steps} iterations")


# what the vector can come to when it is multiplied some fifty times by a power that is scaled by its trace: d times smaller at each product where all
# eigenvalues are alike, and as large as it was where there is one
MANY_PRODUCTS = [(20, 573440), (40, 606208)]


@pytest.mark.parametrize("n,iterations", MANY_PRODUCTS)
def test_flat_spectrum_and_one_eigenvalue_under_many_products(gpu, n, iterations):
    torch, binding = gpu
    print(f"many products n={n} iterations={iterations}", flush=True)
    d = m = 1024
    y = torch.zeros((n, m), device="cuda")
    with binding.EF21(n, d, 1, 0.1) as h:
        A = 32.0 * torch.eye(d, device="cuda").expand(n, m, d).contiguous()         # G = I, and powers of two all the way
        h.set_problem_dense(A, y, 0.0)
        gamma, L, L_i = h.theory_stepsize(iterations)
        np.testing.assert_allclose(list(L_i) + [L], 0.25, rtol=1e-13)
        assert np.isfinite(gamma)
        A.fill_(0.999)                                                              # rank one, its eigenvalue just below 1024
        _, L, L_i = h.theory_stepsize(iterations)
        # fp32 entries of G
        np.testing.assert_allclose(list(L_i) + [L], 0.25 * d * float(np.float32(0.999)) ** 2, rtol=2.0 ** -23)


# n, d (as many rows), the way and the numbers of iterations that go it: each form of the kernels, by columns (three to five per lane of the
# resident one, a launch per step beyond), past a launch's 4096 iterations where the matrices' powers would take too much memory, and by squaring
# at the ends of groups and strips with exponents of few and many bits
REACHED = [
    (48, 192, "iteration", (3, 7, 47)), (48, 192, "recurrence", (48, 100, 177)),
    (48, 256, "iteration", (7, 47)), (48, 256, "recurrence", (48, 177, 178)),
    (60, 320, "iteration", (7, 47)), (60, 320, "recurrence", (48, 178, 400)),
    (48, 700, "iteration", (20, 47)), (48, 700, "recurrence", (48, 177, 178, 400)),
    (48, 1023, "iteration", (40, 2823)), (48, 1023, "recurrence", (48, 178, 1000, 2822)),
    (1300, 192, "iteration", (2823, 4096, 4097)), (700, 256, "iteration", (4096, 4097, 8300)), (450, 300, "iteration", (4096, 4097, 8300)),
    (1, 129, "squaring", (100, 128, 129, 257, 1001)), (3, 143, "squaring", (100, 128, 129, 1001)), (2, 145, "squaring", (100, 128, 129, 1001)),
    (4, 176, "squaring", (100, 128, 257, 1001)), (2, 209, "squaring", (100, 128, 129, 1001)), (2, 305, "squaring", (2, 65, 128, 129, 1001)),
    (2, 320, "squaring", (2, 65, 128, 257, 1001)), (3, 337, "squaring", (65, 128, 129, 1001)), (2, 500, "squaring", (65, 128, 257, 1001)),
    (1, 1009, "squaring", (65, 128, 129, 1001)), (2, 1024, "squaring", (65, 128, 257, 1001)),
]


def spread_eigenvalues(n, d, rng):
    """[n][d] singular values: one eigenvalue of 1, many just below it, at distances for which 48 to a thousand iterations count."""
    scale = rng.random((n, d)).astype(np.float32)
    for row in range(n):
        close = rng.permutation(d)[:d // 2]
        scale[row, close] = 1.0 - 0.5 * rng.choice([0.02, 0.005, 0.002, 0.0005], close.size)
        scale[row, close[0]] = 1.0
    return scale


def estimates(eigenvalues, steps):
    """As diagonal_power, all rows at once: the eigenvalues' powers by logarithms (at 8300 iterations good to 1e-12)."""
    v = np.array([start_vector(eigenvalues.shape[1], row) for row in range(eigenvalues.shape[0])])
    top = eigenvalues.max(1, keepdims=True)
    y = v * np.exp((steps - 1) * np.log(eigenvalues / top))
    return np.linalg.norm(eigenvalues * y, axis=1) / np.linalg.norm(y, axis=1)


@pytest.mark.parametrize("n,d,way,iterations", REACHED)
def test_each_way_gives_the_power_iterations_value(gpu, n, d, way, iterations):
    torch, binding = gpu
    print(f"{way} n={n} d={d}", flush=True)
    scale = spread_eigenvalues(n, d, np.random.default_rng(n + d)) * np.float32(np.sqrt(d))
    A = torch.diag_embed(to_gpu(torch, scale))              # A_i^T A_i / m diagonal: one product per entry, exact in fp64
    diagonals = scale.astype(np.float64) ** 2 / d
    rounded = np.vstack([diagonals, diagonals.mean(0)]).astype(np.float32).astype(np.float64)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(A, torch.zeros((n, d), device="cuda"), 0.0)
        for steps in iterations:
            _, L, L_i = h.theory_stepsize(steps)
            got = 4.0 * np.array(list(L_i) + [L])
            # fp64 on both sides from the same fp32 matrix; the start vectors may differ, see test_recurrence_gives_the_power_iterations_value,
            # and the fewer the iterations the wider the eigenvalues that count: all of them, at most
            rtol = 2.4e-8 if steps >= 48 else 2.0 ** -23
            want = estimates(rounded, steps)
            np.testing.assert_allclose(got, want, rtol=rtol, err_msg=f"{steps} iterations")
            if steps <= 1001:                               # one iteration more or less would show, in the workers' values
                for other in (steps - 1, steps + 1):
                    assert np.median(np.abs(estimates(rounded, other) / want - 1.0)[:n]) > 2 * rtol, (steps, other)


def test_without_memory_for_the_powers_the_matrices_are_used(gpu):
    """Squaring takes 24 bytes per entry of the matrices, the recurrence four and their tiles: 403 and 133 MB here.  With 250 MB left on the card a
    call goes by the recurrence, not back to a thousand passes over A, and the next one in the workspace that is there."""
    torch, binding = gpu
    n, d, iterations = 15, 1024, 1000
    scale = spread_eigenvalues(n, d, np.random.default_rng(5)) * np.float32(np.sqrt(d))
    A = torch.diag_embed(to_gpu(torch, scale))
    diagonals = scale.astype(np.float64) ** 2 / d
    rounded = np.vstack([diagonals, diagonals.mean(0)]).astype(np.float32).astype(np.float64)
    with binding.EF21(n, d, 1, 0.1) as h:
        h.set_problem_dense(A, torch.zeros((n, d), device="cuda"), 0.0)

        def call(steps):
            before = torch.cuda.mem_get_info()[0]
            _, L, L_i = h.theory_stepsize(steps)
            np.testing.assert_allclose(4.0 * np.array(list(L_i) + [L]), estimates(rounded, steps), rtol=2.4e-8)
            taken = before - torch.cuda.mem_get_info()[0]
            print(f"{steps} iterations, {before >> 20} MB there, {taken >> 20} taken", flush=True)
            return taken
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        hogs = []
        try:
            for _ in range(5):                              # one large one leaves more than was asked for
                free = torch.cuda.mem_get_info()[0]
                if free > 270 << 20:
                    hogs.append(torch.empty(free - (250 << 20), dtype=torch.uint8, device="cuda"))
            assert 150 << 20 < torch.cuda.mem_get_info()[0] < 350 << 20
            assert 90 << 20 < call(iterations) < 160 << 20          # of 127; the runtime has some megabytes of its own
            assert call(iterations) < 8 << 20
            assert call(100) < 8 << 20
        finally:
            hogs.clear()
            torch.cuda.empty_cache()
        assert 200 << 20 < call(iterations) < 320 << 20         # by squaring again: the larger workspace for the smaller one
