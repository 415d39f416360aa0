"""The one-launch iteration of small dense problems (ef21_step with EF21_ONE_LAUNCH): bit for bit the
state and the messages of the separate gradient, Top-k and aggregation kernels, step after step, in both loop
orders and for both losses; and against the CPU oracle through f(x^t) (1e-4) and the first message."""
import numpy as np
import pytest

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


def problem(n, d, m, seed):
    rng = np.random.default_rng(seed)
    A = (rng.standard_normal((n, m, d)) / np.sqrt(d)).astype(np.float32)
    w = rng.standard_normal(d)
    y = np.sign(A.astype(np.float64) @ w + 1e-30).astype(np.float32)
    return A, y, rng


SHAPES = [(4, 100, 250, 3),      # the smallest configuration: vec4, one quarter-wave of columns
          (3, 256, 37, 5),       # vec4, a full wavefront of float4
          (2, 333, 41, 4),       # scalar columns, ragged
          (5, 1024, 301, 16),    # the widest rows the kernel takes
          (20, 123, 1628, 1),    # the shape of the paper's a9a split over 20 workers, Top-1
          (7, 68, 1579, 2),      # phishing over 7 workers
          (1, 1, 1, 1),
          (3, 512, 9, 512)]      # k = d


@pytest.mark.parametrize("n,d,m,k", SHAPES)
@pytest.mark.parametrize("order", ["grad_first", "step_first"])
def test_same_bits_as_the_separate_kernels(gpu, n, d, m, k, order):
    torch, binding = gpu
    print(f"one-launch iteration n={n} d={d} m={m} k={k} {order}", flush=True)
    A, y, rng = problem(n, d, m, d + m)
    Ag, yg = to_gpu(torch, A), to_gpu(torch, y)
    x0 = to_gpu(torch, 0.1 * rng.standard_normal(d))
    flag = binding.ORDER_STEP_FIRST if order == "step_first" else binding.ORDER_GRAD_FIRST
    with binding.EF21(n, d, k, 0.5) as one, binding.EF21(n, d, k, 0.5) as sep:
        for h in (one, sep):
            h.set_problem_dense(Ag, yg, 0.1)
            h.set_state(x0, 0.5 * h.local_grad(x0), None)
        for t in range(12):
            one.step(None, flag | binding.ONE_LAUNCH)
            sep.step(None, flag)
            a, b = one.get_state(), sep.get_state()
            for name, u, v in zip(("x", "g_i", "g"), a, b):
                assert torch.equal(u, v), f"step {t}: {name} differs"
            (ia, va), (ib, vb) = one.get_messages(), sep.get_messages()
            assert torch.equal(ia, ib) and torch.equal(va, vb), f"step {t}: messages differ"
        one.set_timing(True)
        one.step(None, flag | binding.ONE_LAUNCH)
        classes = one.get_timing(reset=True)
        one.set_timing(False)
        assert "small_step" in classes and "topk_row" not in classes and "grad_main" not in classes


# a workgroup per worker: every form of its rows (tiny, quads, ragged; 16, 32 and 64 lanes, two quads per lane) with the most rows
# it takes, one row more (the separate kernels), a row or two, and trips that end inside a wavefront's rows
@pytest.mark.parametrize("d", [1, 3, 4, 5, 63, 64, 65, 126, 128, 129, 255, 256, 258, 511, 512, 513])
@pytest.mark.parametrize("loss", ["logistic", "squares"])
def test_workgroup_per_worker(gpu, oracle, d, loss):
    torch, binding = gpu
    most = 512 if d <= 128 else 256 if d <= 256 else 128            # rows: two trips of sixteen wavefronts
    for m in sorted({1, 2, 17, most // 4 - 1, most - 1, most, most + 1}):
        print(f"workgroup per worker d={d} m={m} {loss}", flush=True)
        n, k = 3, max(1, d // 3)
        A, y, rng = problem(n, d, m, d + m)
        if loss == "squares":
            y = rng.standard_normal((n, m)).astype(np.float32)
        x = (0.3 * rng.standard_normal(d)).astype(np.float32)
        batch = rng.integers(0, m, (n, m)).astype(np.int32)
        batch[0, 0], batch[1, m - 1] = -1, m                      # entries that name no row
        P = (oracle.LeastSquaresDense if loss == "squares" else oracle.LogRegDense)(A, y, 0.1)
        with binding.EF21(n, d, k, 0.3) as h, binding.EF21(n, d, k, 0.3) as given:
            for e in (h, given):
                e.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.1)
                if loss == "squares":
                    e.set_loss(binding.LOSS_LEAST_SQUARES)
                e.set_state(to_gpu(torch, x), to_gpu(torch, 0.1 * rng.standard_normal((n, d)) if e is h else h.get_state()[1].cpu()),
                            None)
            got = h.local_grad().cpu().numpy().astype(np.float64)
            ref = P.grads(x.astype(np.float64))
            # per row: the margin's rounding, (d / 64 + 8) u sum |a x| (d / 64 additions per lane, six levels over the lanes), moves
            # the coefficient by at most its curvature (1/4, or 2); sums of at most sixteen levels; helpers.gradient_rounding_floor
            # is the same for the logistic loss
            u = 2.0 ** -24
            a64, z = A.astype(np.float64), np.einsum("imd,d->im", A.astype(np.float64), x.astype(np.float64))
            coef = np.abs(2.0 * (z - y)) if loss == "squares" else 1.0 / (1.0 + np.exp(y * z))
            dz = (d / 64 + 8) * u * np.einsum("imd,d->im", np.abs(a64), np.abs(x.astype(np.float64)))
            dcoef = (2.0 if loss == "squares" else 0.25) * dz + 16 * u * (coef + (2.0 * np.abs(z) if loss == "squares" else 0.0))
            bound = 1e-6 * np.abs(ref) + np.einsum("imd,im->id", np.abs(a64), dcoef) / m + u
            assert np.all(np.abs(got - ref) <= bound), (m, np.max(np.abs(got - ref) / bound))
            for rows in (None, to_gpu(torch, batch, np.int32)):
                h.set_minibatch(rows)
                given.set_minibatch(rows)
                for _ in range(2):                                # its lines 5 and 6 against the Top-k of the reported gradient
                    s = given.local_grad()
                    h.step()
                    given.step(s)
                    for name, a, b in zip(("x", "g_i", "g"), h.get_state(), given.get_state()):
                        assert torch.equal(a, b), f"m = {m}: {name} differs"
                    for a, b in zip(h.get_messages(), given.get_messages()):
                        assert torch.equal(a, b), f"m = {m}: messages differ"


@pytest.mark.parametrize("n", [256, 257])
def test_workgroup_per_worker_up_to_the_compute_units(gpu, oracle, n):
    """One workgroup per worker where each has a compute unit to itself; with more workers they take turns and an iteration is
    slower than by the separate kernels (n = 257, m = 20, d = 500: 36.0 and 33.9 us).  One launch, the separate kernels
    and an iteration from the reported gradient agree bit for bit on either side."""
    torch, binding = gpu
    d, m, k = 60, 20, 2
    A, y, rng = problem(n, d, m, n)
    x, g_i = (0.3 * rng.standard_normal(d)).astype(np.float32), 0.1 * rng.standard_normal((n, d))
    P = oracle.LogRegDense(A, y, 0.1)
    with binding.EF21(n, d, k, 0.3) as own, binding.EF21(n, d, k, 0.3) as given, binding.EF21(n, d, k, 0.3) as one:
        for h in (own, given, one):
            h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.1)
            h.set_state(to_gpu(torch, x), to_gpu(torch, g_i), None)
        s = own.local_grad()
        # as in test_workgroup_per_worker
        u = 2.0 ** -24
        a64, x64 = A.astype(np.float64), x.astype(np.float64)
        coef = 1.0 / (1.0 + np.exp(y * np.einsum("imd,d->im", a64, x64)))
        dcoef = 0.25 * (d / 64 + 8) * u * np.einsum("imd,d->im", np.abs(a64), np.abs(x64)) + 16 * u * coef
        ref = P.grads(x64)
        bound = 1e-6 * np.abs(ref) + np.einsum("imd,im->id", np.abs(a64), dcoef) / m + u
        assert np.all(np.abs(s.cpu().numpy() - ref) <= bound)
        for t in range(3):
            given.step(given.local_grad())
            one.step(None, binding.ONE_LAUNCH)
            if t == 2:
                own.set_timing(True)
            own.step()
            for h in (given, one):
                for a, b in zip(own.get_state() + own.get_messages(), h.get_state() + h.get_messages()):
                    assert torch.equal(a, b), f"step {t}"
        assert ("topk_row" in own.get_timing()) == (n > 256)       # beyond, a Top-k kernel of its own


def test_least_squares_same_bits(gpu):
    torch, binding = gpu
    n, d, m, k = 3, 200, 90, 7
    A, _, rng = problem(n, d, m, 5)
    b = rng.standard_normal((n, m)).astype(np.float32)
    Ag, bg = to_gpu(torch, A), to_gpu(torch, b)
    x0 = torch.zeros(d, device="cuda")
    with binding.EF21(n, d, k, 0.2) as one, binding.EF21(n, d, k, 0.2) as sep:
        for h in (one, sep):
            h.set_problem_dense(Ag, bg, 0.0)
            h.set_loss(binding.LOSS_LEAST_SQUARES)
            h.set_state(x0, torch.zeros((n, d), device="cuda"), None)
        for t in range(10):
            one.step(None, binding.ONE_LAUNCH)
            sep.step()
            for u, v in zip(one.get_state(), sep.get_state()):
                assert torch.equal(u, v), f"step {t}"


def test_against_the_oracle(gpu, oracle):
    torch, binding = gpu
    n, d, m, k = 4, 100, 250, 3
    A, y, rng = problem(n, d, m, 6)
    P = oracle.LogRegDense(A, y, 0.1)
    gamma = float(np.float32(0.5))
    x0 = np.zeros(d)
    st = oracle.init_state(x0, P.grads(x0), k, init="zero", storage_f32=True)
    with binding.EF21(n, d, k, gamma) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.1)
        h.set_state(to_gpu(torch, st.x), to_gpu(torch, st.g_i), to_gpu(torch, st.g))
        grads0 = h.local_grad(None).cpu().numpy()
        f0 = P.loss(x0)
        for t in range(60):
            oracle.iteration(st, P.grads, k, gamma)
            h.step(None, binding.ONE_LAUNCH)
            if t == 0:        # zero state: the message is the Top-k of the gradient the library itself reports
                idx, val = h.get_messages()
                ref_idx, ref_val = oracle.topk_rows(grads0.astype(np.float64), k)
                assert np.array_equal(idx.cpu().numpy(), ref_idx)
                assert np.array_equal(val.cpu().numpy(), ref_val.astype(np.float32))
            f_ref, f_gpu = P.loss(st.x), P.loss(h.get_x().cpu().numpy().astype(np.float64))
            assert abs(f_gpu - f_ref) <= 1e-4 * abs(f_ref), f"iteration {t}: {f_gpu} vs {f_ref}"
        assert f_ref < f0


def test_larger_problems_keep_the_separate_kernels(gpu):
    torch, binding = gpu
    n, d, m, k = 2, 2000, 40, 5          # d above the one-launch limit
    A, y, _ = problem(n, d, m, 7)
    with binding.EF21(n, d, k, 0.5) as h:
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.1)
        h.set_timing(True)
        h.step(None, binding.ONE_LAUNCH)
        classes = h.get_timing(reset=True)
        assert "small_step" not in classes and "grad_main" in classes
    with binding.EF21(4, 100, 3, 0.5) as h:          # and a qualifying problem takes them unless asked
        A, y, _ = problem(4, 100, 250, 8)
        h.set_problem_dense(to_gpu(torch, A), to_gpu(torch, y), 0.1)
        h.set_timing(True)
        h.step()
        classes = h.get_timing(reset=True)
        assert "small_step" not in classes and "grad_main" in classes


def test_flag_combinations(gpu):
    torch, binding = gpu
    with binding.EF21(2, 16, 2, 0.1) as h:
        g = torch.ones((2, 16), device="cuda")
        h.step(g, binding.ONE_LAUNCH)                      # supplied gradients: the flag changes nothing
        h.step(g, binding.ONE_LAUNCH | binding.PLUS | binding.ORDER_STEP_FIRST)
        h.step(g, binding.ONE_LAUNCH | binding.CLASSIC_EF)
        for bad in (16, binding.CLASSIC_EF | binding.PLUS, binding.CLASSIC_EF | binding.ORDER_STEP_FIRST):
            with pytest.raises(binding.EF21Error):
                h.step(g, bad)
