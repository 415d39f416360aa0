"""GPU parity of the batched Top-k (ef21_topk through the C ABI) against the CPU oracle:
positions bit-exact, values bit-exact (they are copies of the inputs)."""
import numpy as np
import pytest

from helpers import best_time, same_bits, sampled_positions
from paper_2106_05203_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2106_05203_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load_library()
    return torch, binding


def run_gpu(gpu, V, k):
    torch, binding = gpu
    t = torch.from_numpy(np.ascontiguousarray(V, dtype=np.float32)).cuda()
    idx, val = binding.ef21_topk(t, k)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), val.cpu().numpy()


def check(gpu, oracle, V, k, rows=None):
    print(f"topk case n={V.shape[0]} d={V.shape[1]} k={k}", flush=True)
    idx, val = run_gpu(gpu, V, k)
    rows = range(V.shape[0]) if rows is None else rows
    for i in rows:
        ref_idx, ref_val = oracle.topk(V[i].astype(np.float64), k)
        assert np.array_equal(idx[i], ref_idx), f"row {i}: positions differ"
        assert same_bits(val[i], ref_val.astype(np.float32)), f"row {i}: values differ"
    # properties that hold for every row at any size
    assert np.all(np.diff(idx.astype(np.int64), axis=1) > 0)
    assert np.all((idx >= 0) & (idx < V.shape[1]))
    assert same_bits(val, np.take_along_axis(V, idx.astype(np.int64), axis=1))
    return idx, val


def test_tiny_patterns(gpu, oracle):
    pats = [
        [0.0], [-3.0], [0.0, 0.0, 0.0, 0.0], [0.0, -0.0, 0.0, -0.0, 1.0],
        [1.0, -1.0, 1.0, -1.0, 1.0], [3, -5, 1, 5, -2], [5, 4, 3, 2, 1, 0, -1, -2, -3, -4, -5],
        [1e-45, -1e-45, 0.0, 2e-45], [np.inf, -np.inf, 1.0, 3e38],
    ]
    for v in pats:
        v = np.array(v, dtype=np.float32)
        for k in range(1, v.size + 1):
            check(gpu, oracle, v[None, :].repeat(3, axis=0), k)


@pytest.mark.parametrize("d", [1, 2, 63, 64, 65, 127, 1000, 1023, 1024, 1025, 4096, 5000, 16385, 40000])
def test_random_small_rows(gpu, oracle, d):
    rng = np.random.default_rng(d)
    V = rng.standard_normal((5, d)).astype(np.float32)
    V[1] = np.round(V[1] * 2) / 2                      # heavy ties
    V[2] = 0.0                                         # all equal
    V[3, ::3] = -V[3, (d // 2) % d]                    # one value repeated with flipped sign
    V[4] *= np.float32(1e-41)                          # subnormals
    for k in sorted(k for k in {1, 2, d // 100, d // 2, d - 1, d} if 1 <= k <= d):
        check(gpu, oracle, V, k)


@pytest.mark.parametrize("d", [3, 64, 65, 128, 129, 171, 205, 255, 256])
def test_rows_ranked_whole(gpu, oracle, d):
    """Rows of at most 256 entries, where the comparisons are shared among 1024 // d threads an entry: ties across the
    threads' and the wavefronts' shares, infinities, and every fifth k."""
    rng = np.random.default_rng(d)
    V = rng.integers(-3, 4, size=(3, d)).astype(np.float32)
    V[1] = rng.standard_normal(d).astype(np.float32)
    V[1, rng.integers(0, d, size=d // 8 + 1)] = np.inf
    V[2] = np.where(rng.random(d) < 0.5, -0.25, 0.25).astype(np.float32)
    for k in sorted({1, 2, d - 1, d} | set(range(1, d, 5))):
        check(gpu, oracle, V, k)


@pytest.mark.parametrize("d", [200, 256, 257, 5000, 9000, 300_000])
@pytest.mark.parametrize("crowd", [3, 255, 256, 257, 600])
def test_threshold_inside_a_bin_of_near_equal_magnitudes(gpu, oracle, d, crowd):
    """`crowd` entries share the twelve leading key bits (values in [1, 1.0625), many of them exactly equal up
    to sign), a few are larger, the rest tiny; k runs through the crowd, so the threshold key and the tie quota
    are decided among them: by ranking them directly up to 256, by further histogram passes beyond."""
    crowd = min(crowd, d - 2)
    rng = np.random.default_rng(d * 1000 + crowd)
    V = (1e-4 * rng.standard_normal((4, d))).astype(np.float32)
    for i in range(4):
        pos = rng.choice(d, size=crowd + 2, replace=False)
        vals = 1.0 + rng.integers(0, 8, size=crowd) / 128.0            # 8 distinct magnitudes: heavy ties
        V[i, pos[:crowd]] = (vals * rng.choice([-1.0, 1.0], size=crowd)).astype(np.float32)
        V[i, pos[crowd:]] = [3.0, -2.5]
    for k in sorted({1, 2, 3, 2 + crowd // 3, 2 + crowd // 2, 1 + crowd, 2 + crowd, min(d, 3 + crowd)}):
        check(gpu, oracle, V, k)


@pytest.mark.parametrize("d", [16384, 20001, 50000, 61440, 61441])
@pytest.mark.parametrize("k", [1, 37, 1000, 1024, 1025])
def test_rows_held_in_lds_as_key_prefixes(gpu, oracle, d, k):
    """Rows of 16 384 to 61 440 entries with k <= 1024 are selected by one workgroup (by its registers; a kernel with 16 bits
    of every key in LDS before; the sizes around those limits take the other kernels).  Rows: Gaussian; heavy exact ties (the list
    of entries above the bound overflows); a crowded bin of near-equal magnitudes with ties (a second histogram, or
    the bisection); fewer non-zeros than k (the threshold is zero); infinities and a row of one value."""
    rng = np.random.default_rng(d + k)
    V = rng.standard_normal((7, d)).astype(np.float32)
    V[1] = np.round(V[1] * 2) / 2
    V[2] = (1e-3 * rng.standard_normal(d)).astype(np.float32)
    crowd = rng.choice(d, size=3000, replace=False)
    V[2, crowd] = ((1.0 + rng.integers(0, 2000, size=3000) / 32768.0) * rng.choice([-1.0, 1.0], size=3000)).astype(np.float32)
    V[3] = 0.0
    few = rng.choice(d, size=min(k, 700) // 2 + 1, replace=False)
    V[3, few] = rng.standard_normal(few.size).astype(np.float32)
    V[4, rng.choice(d, size=5, replace=False)] = [np.inf, -np.inf, 3e38, -3e38, np.inf]
    V[5] = -2.5
    V[6] = (rng.standard_t(3, size=d) * 1e-3).astype(np.float32)
    check(gpu, oracle, V, k)


def rows_for_registers(d, k, seed):
    """One row per way through the kernel that holds the row in registers: an ordinary one, ties everywhere, fewer than k
    non-zeros, magnitudes all alike (the list or the threshold's bin overflows), large entries side by side, a threshold far
    above the bound (beyond the window), NaN and infinities, large entries at the row's very end, entries piled up."""
    rng = np.random.default_rng(seed)
    V = rng.standard_normal((9, d)).astype(np.float32)
    V[1] = np.round(V[1] * 2) / 2
    V[2] = np.where(rng.random(d) < 0.5 * k / d, V[2], np.where(V[2] > 0, 0.0, -0.0))
    V[3] = 10 + 0.01 * V[3]
    V[4, d // 3:d // 3 + min(2 * k, d // 4)] *= 100
    V[5, ::7] *= np.exp(20 * rng.random(V[5, ::7].size)).astype(np.float32)
    V[6, ::d // 5] = np.nan
    V[6, 1::d // 3] = np.inf
    V[7, -3:] = [1e30, -1e30, 1e30]
    V[8] = np.sign(V[8]) * (1 - 5e-4 * rng.random(d))          # piled up: more than 256 entries in T's bin, few within four keys
    return V.astype(np.float32)


def first_by_magnitude(V, k):
    """Ascending positions of the k largest magnitude keys, ties to the lower position (NaN above infinity, as the
    kernels order the bits)."""
    key = (V.view(np.int32) & 0x7fffffff).astype(np.int64)
    return np.sort(np.argsort(-key, axis=1, kind="stable")[:, :k], axis=1)


@pytest.mark.parametrize("d", [512, 513, 1025, 4095, 4096, 4097, 8192, 8195, 12289, 16385, 24577, 36865, 53249, 61439, 61440])
def test_rows_held_in_registers(gpu, d):
    """The edges of every length of the register array (4096 entries a quad), k up to its limits."""
    for k in sorted({1, max(1, d // 100), min(d // 8, 1024)}):
        V = rows_for_registers(d, k, d + k)
        idx, val = run_gpu(gpu, V, k)
        ref = first_by_magnitude(V, k)
        assert np.array_equal(idx, ref), (d, k)
        assert same_bits(val, np.take_along_axis(V, ref, axis=1)), (d, k)


@pytest.mark.parametrize("n", [9, 261])
@pytest.mark.parametrize("d", [511, 512, 799, 800, 1023, 1024])
def test_either_side_of_the_shortest_rows_in_registers(gpu, n, d):
    """The shortest rows that go there depend on whether there are more of them than compute units."""
    for k in (1, d // 20, d // 8):
        V = np.tile(rows_for_registers(d, k, d + k), (n // 9, 1))
        idx, val = run_gpu(gpu, V, k)
        ref = first_by_magnitude(V, k)
        assert np.array_equal(idx, ref), (n, d, k)
        assert same_bits(val, np.take_along_axis(V, ref, axis=1)), (n, d, k)


@pytest.mark.parametrize("copies", [1, 2])
@pytest.mark.parametrize("d", [513, 4097, 12289, 24577, 50001, 61440])
def test_differences_held_in_registers(gpu, d, copies):
    """The same for grad - g_i inside a step: message, g_i updated at the kept positions only, and g and x, which are added
    up by the index that the kernel writes on each of its ways (9 workers: blocks of 512 columns, 18: of 256)."""
    torch, binding = gpu
    k = min(d // 8, 500)
    S = rows_for_registers(d, k, d)
    S[6] = S[0]                                        # (a step keeps NaN in its state: not compared here)
    G = np.random.default_rng(d + 1).standard_normal(S.shape).astype(np.float32)
    G[1:3] = 0.0                                       # ties and zeros stay what they are
    S, G = np.tile(S, (copies, 1)), np.tile(G, (copies, 1))
    n = S.shape[0]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    with binding.EF21(n, d, k, 0.1) as h:
        h.set_state(x=torch.zeros(d, device="cuda"), g_i=dev(G), g=torch.zeros(d, device="cuda"))
        h.step(dev(S))
        idx, val = (t.cpu().numpy() for t in h.get_messages())
        x, g_i, g = (t.cpu().numpy() for t in h.get_state())
    diff = S - G
    ref = first_by_magnitude(diff, k)
    assert np.array_equal(idx, ref)
    kept = np.take_along_axis(diff, ref, axis=1)
    assert same_bits(val, kept)
    want = G.copy()
    np.put_along_axis(want, ref, np.take_along_axis(G, ref, axis=1) + kept, axis=1)
    assert same_bits(g_i, want)
    c = np.zeros((n, d))
    np.put_along_axis(c, ref, kept.astype(np.float64), axis=1)
    # n - 1 additions, the rounding of 1 / n and the fused multiply-add
    assert np.all(np.abs(g - c.mean(axis=0)) <= (n + 2) * 2.0**-24 * np.abs(c).mean(axis=0))
    assert np.array_equal(x, np.float32(-0.1) * g)


@pytest.mark.parametrize("d,k", [(70001, 700), (262144, 5), (300007, 3000), (1_000_003, 999), (70001, 1), (1_000_003, 1),
                                 (262144, 1)])
def test_long_rows_ragged(gpu, oracle, d, k):
    V = workloads.topk_rows(3, d, seed=d % 1000)
    check(gpu, oracle, V, k)
    W = workloads.force_threshold_ties(V, k, copies=8, seed=1)
    check(gpu, oracle, W, k)


def test_long_rows_degenerate(gpu, oracle):
    d = 200_000
    V = np.zeros((4, d), dtype=np.float32)
    V[1] = 1.5
    V[1, ::2] = -1.5
    V[2, 1000:] = np.float32(2.0) ** -130               # subnormal plateau
    V[3] = np.arange(d, dtype=np.float32)[::-1]
    for k in (1, 777, d // 2, d):
        check(gpu, oracle, V, k)


@pytest.mark.parametrize("k", [10000, 60000])
def test_long_rows_misleading_sample(gpu, oracle, k):
    """The long-row path guesses a candidate threshold from 64 evenly spaced pieces of 64 entries.
    Here the large values sit exactly on those pieces and nowhere else, so the guess keeps far fewer
    than k candidates and the exact per-row algorithm has to take over (both the small-k and the
    large-k variant of the candidate stage)."""
    d = 300_000
    rng = np.random.default_rng(k)
    V = (rng.standard_normal((3, d)) * 1e-3).astype(np.float32)
    pos = sampled_positions(d)
    V[:, pos] = (1.0 + rng.random((3, pos.size))).astype(np.float32)
    V[2] = np.abs(V[2])
    check(gpu, oracle, V, k)


@pytest.mark.parametrize("k", [10000, 60000])
def test_long_rows_sample_far_too_low(gpu, oracle, k):
    """The opposite mistake: the sampled pieces hold tiny values and everything else is large, so the
    guessed threshold admits every entry and the k-th largest magnitude lies far above it (above the
    window of leading digits the collect pass counts, for the large-k variant).  Same results."""
    d = 300_000
    rng = np.random.default_rng(k + 1)
    V = (1000.0 * (1.0 + rng.random((3, d)))).astype(np.float32)
    pos = sampled_positions(d)
    V[:, pos] = (rng.standard_normal((3, pos.size)) * 1e-3).astype(np.float32)
    V[1] = -V[1]
    check(gpu, oracle, V, k)


@pytest.mark.parametrize("n,d,k", [(2, 1_500_000, 100_000), (1, 2_000_001, 700_000), (3, 400_000, 399_999)])
def test_long_rows_large_k(gpu, oracle, n, d, k):
    """k large enough that the candidates are processed by many workgroups per row."""
    V = workloads.topk_rows(n, d, seed=k % 97)
    check(gpu, oracle, V, k)
    check(gpu, oracle, workloads.force_threshold_ties(V, k, copies=8, seed=3), k)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("k", [1, 1000, 10000])
def test_config1_full_size(gpu, oracle, k):
    """n = 20 rows of 10^6 N(0,1) values with 1 % exact duplicates (+a / -a), the size the
    throughput is quoted on, and the variant whose threshold magnitude is tied."""
    V = workloads.topk_rows(20, 1_000_000, seed=0)
    check(gpu, oracle, V, k)
    W = workloads.force_threshold_ties(V[:4], k, copies=8, seed=2)
    check(gpu, oracle, W, k)


def test_random_shapes(gpu, oracle):
    """Sixty seeded draws of (n, d, k, kind of row) across all the kernels' ranges of d and k."""
    rng = np.random.default_rng(2106)
    for case in range(60):
        d = int(np.exp(rng.uniform(0.0, np.log(400_000))))
        n = int(rng.integers(1, 5))
        k = int(min(d, max(1, [1, 2, rng.integers(1, 64), d // 100 + 1, d // 3 + 1, d][rng.integers(0, 6)])))
        kind = int(rng.integers(0, 5))
        if kind == 0:
            V = rng.standard_normal((n, d))
        elif kind == 1:
            V = np.round(rng.standard_normal((n, d)) * 3) / 3          # heavy ties
        elif kind == 2:
            V = rng.standard_t(2, size=(n, d)) * 1e-4                  # heavy tails
        elif kind == 3:
            V = np.zeros((n, d))
            nz = rng.integers(0, d, size=max(1, d // 50))
            V[:, nz] = rng.standard_normal((n, nz.size))               # mostly zeros
        else:
            V = np.exp(rng.uniform(-80, 80, size=(n, d))) * rng.choice([-1.0, 1.0], size=(n, d))   # all exponents
        check(gpu, oracle, V.astype(np.float32), k)


def test_deterministic(gpu):
    torch, binding = gpu
    V = torch.from_numpy(workloads.topk_rows(6, 300_000, seed=9)).cuda()
    a = binding.ef21_topk(V, 3000)
    b = binding.ef21_topk(V, 3000)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))


def test_error_codes(gpu):
    torch, binding = gpu
    V = torch.zeros((2, 10), device="cuda")
    for k in (0, 11):
        with pytest.raises(binding.EF21Error) as e:
            binding.ef21_topk(V, k)
        assert e.value.code == binding.EF21_EINVAL
    with pytest.raises(TypeError):
        binding.ef21_topk(V.double(), 1)


def test_calls_on_two_streams_overlap_safely(gpu, oracle):
    """ef21_topk keeps one workspace per stream: calls enqueued on two streams without any ordering between them
    (long rows, so both use a workspace) must each give their own input's selection."""
    torch, binding = gpu
    n, d, k = 6, 400_000, 4000
    A = torch.from_numpy(workloads.topk_rows(n, d, seed=21)).cuda()
    B = torch.from_numpy(workloads.topk_rows(n, d, seed=22)).cuda()
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for rep in range(6):
        with torch.cuda.stream(s1):
            ia, va = binding.ef21_topk(A, k)
        with torch.cuda.stream(s2):
            ib, vb = binding.ef21_topk(B, k + rep)
        outs.append((ia, va, ib, vb))
    torch.cuda.synchronize()
    ref_a = oracle.topk(A[2].cpu().numpy().astype(np.float64), k)
    for rep, (ia, va, ib, vb) in enumerate(outs):
        assert np.array_equal(ia[2].cpu().numpy(), ref_a[0]) and same_bits(va[2].cpu().numpy(), ref_a[1].astype(np.float32))
        ref_b = oracle.topk(B[4].cpu().numpy().astype(np.float64), k + rep)
        assert np.array_equal(ib[4].cpu().numpy(), ref_b[0]) and same_bits(vb[4].cpu().numpy(), ref_b[1].astype(np.float32))
        assert same_bits(va.cpu().numpy(), np.take_along_axis(A.cpu().numpy(), ia.cpu().numpy().astype(np.int64), axis=1))
        assert same_bits(vb.cpu().numpy(), np.take_along_axis(B.cpu().numpy(), ib.cpu().numpy().astype(np.int64), axis=1))


@pytest.mark.parametrize("kind", ["equal", "distinct"])
def test_crowded_threshold_bin_on_long_rows(gpu, oracle, kind):
    """Thousands of candidates share the histogram bin of the threshold: 6000 copies of one magnitude (no ranking
    needed: ties go to the lower positions), or 6000 consecutive floats (too many to rank: the exact per-row
    algorithm takes over).  k is chosen so that the threshold falls inside the cluster."""
    rng = np.random.default_rng(8)
    n, d = 3, 250_000
    V = (0.1 * rng.standard_normal((n, d))).astype(np.float32)
    for i in range(n):
        pos = rng.choice(d, size=6000, replace=False)
        if kind == "equal":
            V[i, pos] = np.where(rng.random(6000) < 0.5, 1.0, -1.0).astype(np.float32)
        else:
            bits = np.float32(1.0).view(np.uint32) + rng.permutation(6000).astype(np.uint32)
            V[i, pos] = bits.view(np.float32) * np.where(rng.random(6000) < 0.5, 1.0, -1.0).astype(np.float32)
    for k in (3000, 5999, 6001):
        check(gpu, oracle, V, k)


# rows at an odd 4-byte address and of lengths that leave one, two and three entries after the last whole load, on both
# sides of every limit that chooses piece length (two million entries in all) and bin width (k = 4096, k = 131072 with
# less than one entry in 200 kept, k = 400000), and the LDS copies of the row kernel (8192, 16384)
@pytest.mark.parametrize("n,d,k", [(2, 8193, 82), (3, 16383, 1025), (3, 16386, 4096), (3, 16387, 4097), (2, 999_999, 4097),
                                   (2, 1_000_001, 4096), (1, 1_000_003, 400_000), (1, 1_000_003, 400_001), (3, 70_002, 1),
                                   (1, 2_000_517, 9_000), (1, 30_000_001, 131_073)])
def test_rows_at_any_address(gpu, oracle, n, d, k):
    torch, binding = gpu
    print(f"unaligned topk case n={n} d={d} k={k}", flush=True)
    rng = np.random.default_rng(d + k)
    V = rng.standard_t(3, size=(n, d)).astype(np.float32) if d < 10_000_000 else rng.standard_normal((n, d), dtype=np.float32)
    V[:, ::7] = np.round(V[:, ::7] * 8) / 8                                  # ties
    pad = torch.empty(n * d + 1, device="cuda")
    rows = pad[1:].view(n, d)
    rows.copy_(torch.from_numpy(V))
    idx, val = (t.cpu().numpy() for t in binding.ef21_topk(rows, k))
    for i in range(n):
        key = np.abs(V[i])
        order = np.argsort(-key, kind="stable")[:k] if d < 10_000_000 else None
        if order is None:                                                    # the same selection without a full sort
            T = np.partition(key, d - k)[d - k]
            above = np.nonzero(key > T)[0]
            order = np.concatenate([above, np.nonzero(key == T)[0][:k - above.size]])
        want = np.sort(order)
        assert np.array_equal(idx[i], want), f"row {i}: positions differ"
        assert same_bits(val[i], V[i][want])


def to_gpu(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def largest(V, k):
    """Positions (ascending) of the k largest magnitudes of one row, ties to the lower position, without a full sort."""
    key = np.abs(V)
    T = np.partition(key, key.size - k)[key.size - k]
    above = np.nonzero(key > T)[0]
    return np.sort(np.concatenate([above, np.nonzero(key == T)[0][:k - above.size]]))


def rows_like(kind, rng, n, d):
    if kind == "uniform":
        return rng.random((n, d), dtype=np.float32)
    if kind == "offset":
        return np.float32(10) + np.float32(0.02) * rng.standard_normal((n, d), dtype=np.float32)
    if kind == "student":
        return rng.standard_t(3, size=(n, d)).astype(np.float32)
    return rng.standard_normal((n, d), dtype=np.float32)


# rows whose largest entries lie close together (many of them in one wide bin of the candidates' histogram), rows with a
# heavy tail (the threshold far above the sample's bound) and Gaussian ones, k on both sides of the limits that choose
# the widest bin: right, and no row by the one-workgroup algorithm, which takes milliseconds for rows this long
@pytest.mark.parametrize("n,d,k", [(1, 3_000_000, 1000), (2, 3_000_000, 4096), (1, 7_000_000, 12_000), (2, 1_000_000, 1000),
                                   (1, 5_000_000, 100)])
def test_flat_and_heavy_rows_take_the_fast_path(gpu, n, d, k):
    torch, binding = gpu
    print(f"flat rows n={n} d={d} k={k}", flush=True)
    rng = np.random.default_rng(d + k)
    V = rows_like("normal", rng, n, d)
    rows = to_gpu(torch, V)
    binding.ef21_topk(rows, k)
    usual = best_time(torch, lambda: binding.ef21_topk(rows, k))
    for kind in ("uniform", "offset", "student"):
        if kind == "offset" and k > 1000:
            continue                                  # more than kTieCap entries at the threshold however narrow the bin
        V = rows_like(kind, rng, n, d)
        rows = to_gpu(torch, V)
        idx, val = (t.cpu().numpy() for t in binding.ef21_topk(rows, k))
        for i in range(n):
            want = largest(V[i], k)
            assert np.array_equal(idx[i], want), f"{kind}, row {i}"
            assert same_bits(val[i], V[i][want]), f"{kind}, row {i}"
        took = best_time(torch, lambda: binding.ef21_topk(rows, k))
        print(f"  {kind}: {took:.0f} us, normal {usual:.0f} us", flush=True)
        assert took <= 12 * usual + 100, f"{kind}: {took:.0f} us against {usual:.0f} us"


@pytest.mark.parametrize("kind", ["uniform", "student"])
@pytest.mark.parametrize("n,d,k", [(2, 5_000_000, 1000), (3, 3_000_000, 9000)])
def test_flat_and_heavy_gradients_take_the_fast_path(gpu, n, d, k, kind):
    """The same inside ef21_step, whose thresholds and bin widths carry over from step to step."""
    torch, binding = gpu
    print(f"flat gradients {kind} n={n} d={d} k={k}", flush=True)
    rng = np.random.default_rng(d + k)
    g_i = np.zeros((n, d), np.float32)
    times = {}
    with binding.EF21(n, d, k, 0.01) as h:
        for what in (kind, "normal"):
            g_i[:] = 0.0
            h.set_state(torch.zeros(d, device="cuda"), to_gpu(torch, g_i))
            pool = [rows_like(what, rng, n, d) for _ in range(2)]
            dev = [to_gpu(torch, v) for v in pool]
            for t in range(4):
                diff = pool[t % 2] - g_i
                h.step(dev[t % 2])
                idx, val = (a.cpu().numpy() for a in h.get_messages())
                for i in range(n):
                    want = largest(diff[i], k)
                    assert np.array_equal(idx[i], want), f"{what}, step {t}, row {i}"
                    assert same_bits(val[i], diff[i][want]), f"{what}, step {t}, row {i}"
                    g_i[i, want] += diff[i][want]
            turn = [0]

            def one():
                turn[0] ^= 1
                h.step(dev[turn[0]])
            times[what] = best_time(torch, one)
    print(f"  {times}", flush=True)
    assert times[kind] <= 12 * times["normal"] + 100, times


# rows just too long for the short LDS copy, as many as there are compute units (the long copy) and more (none)
@pytest.mark.parametrize("n,d,k", [(256, 8193, 80), (257, 8193, 80), (300, 16_383, 1), (513, 9001, 9001), (300, 12_001, 1200)])
def test_many_rows_of_moderate_length(gpu, n, d, k):
    torch, binding = gpu
    print(f"many rows n={n} d={d} k={k}", flush=True)
    rng = np.random.default_rng(d + k)
    V = np.round(rng.standard_normal((n, d), dtype=np.float32) * 64) / 64          # ties
    g_i = np.round(rng.standard_normal((n, d), dtype=np.float32) * 64) / 64
    idx, val = (t.cpu().numpy() for t in binding.ef21_topk(to_gpu(torch, V), k))
    diff = V - g_i
    with binding.EF21(n, d, k, 1.0) as h:
        h.set_state(torch.zeros(d, device="cuda"), to_gpu(torch, g_i))
        h.step(to_gpu(torch, V))
        m_idx, m_val = (t.cpu().numpy() for t in h.get_messages())
        g_new = h.get_state()[1].cpu().numpy()
        h.set_state(torch.zeros(d, device="cuda"), to_gpu(torch, g_i))
        h.step(to_gpu(torch, V), binding.CLASSIC_EF)
        e_idx, e_val = (t.cpu().numpy() for t in h.get_messages())
        e_new = h.get_state()[1].cpu().numpy()
    for i in range(n):
        want = largest(V[i], k)
        assert np.array_equal(idx[i], want) and same_bits(val[i], V[i][want]), f"row {i}"
        want = largest(diff[i], k)
        assert np.array_equal(m_idx[i], want) and same_bits(m_val[i], diff[i][want]), f"row {i}: message"
        row = g_i[i].copy()
        row[want] += diff[i][want]
        assert same_bits(g_new[i], row), f"row {i}: g_i"
        p = g_i[i] + V[i]                                     # exact: multiples of 1/64
        want = largest(p, k)
        assert np.array_equal(e_idx[i], want) and same_bits(e_val[i], p[want]), f"row {i}: EF message"
        p[want] = 0.0
        assert same_bits(e_new[i], p), f"row {i}: error"


def test_rows_just_too_long_for_the_short_copy(gpu):
    """1000 rows of 8193 and of 8192 entries: a workgroup of either takes as much room, so they take as long (with the
    long LDS copy 41 us against 28, so 31)."""
    torch, binding = gpu
    times = {}
    for d in (8192, 8193):
        rows = torch.randn((1000, d), device="cuda")
        times[d] = best_time(torch, lambda: binding.ef21_topk(rows, 81), calls=20)
    print(times, flush=True)
    assert times[8193] <= 1.27 * times[8192], times
