"""The wavefront-update planner against the oracle's stable bucketing: block
starts and planned positions, bit for bit, at the grid sides where the
scatter's block-id width changes (4, 8, 16, 32), for both cuts, for models
narrower than the grid, and at sizes where one of its 512 chunks fills one tile
of 8192 samples, one more, and several; above 2^32 - 1 samples (another variant
of the scatter) against the definition of the order itself.  Then the one-block
grid, which is the caller's array as it stands."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05838_amd import mfsgd
    mfsgd.lib()
    yield mfsgd
    mfsgd.finalize()


def samples(m, n, nnz, seed, skew):
    rng = np.random.default_rng(seed)
    S = np.zeros(nnz, dtype=[("u", "<i4"), ("v", "<i4"), ("r", "<f4")])
    S["u"], S["v"], S["r"] = rng.integers(0, m, nnz), rng.integers(0, n, nnz), rng.random(nnz)
    if skew and nnz:  # half of the samples on one item: equal blocks within one step of 64
        S["v"][::2] = n - 1
    return S


@pytest.mark.parametrize("balance", [0, 1])
@pytest.mark.parametrize("s", [1, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64])
def test_plan_equals_the_oracles_bucketing(M, s, balance):
    M.reset_options()
    M.set_option("balance", balance)
    M.set_option("debug", 1)
    for m, n, nnz in ((4001, 1999, 600_011), (4001, 1999, 8193), (3, 2, 8192), (200_000_033, 7, 1000), (77, 50, 63),
                      (5, 70, 1), (5, 70, 0)):
        if m > 1_000_000 and balance:
            continue  # the balanced cut counts every index
        M.set_option("dtype", 1)
        M.init(m, n, 8, 1)
        S = samples(m, n, nnz, 100 * s + nnz % 97, skew=nnz == 8193)
        if m > 1_000_000:  # indices beyond 24 bits, at both ends of every range
            edges = (np.arange(s + 1, dtype=np.int64) * m + s - 1) // s
            ends = np.concatenate([edges[:-1], edges[1:] - 1]).astype(np.int32)
            S["u"][:len(ends)] = ends
        order, start = oracle.block_order(S, m, n, s, balanced=bool(balance))
        dS = M.samples_to_device(S)
        M.plan(dS, s)
        got = M.debug_plan_starts(s).cpu().numpy()
        assert np.array_equal(got, start), (m, n, nnz)
        assert np.array_equal(M.debug_plan_order(nnz).cpu().numpy(), order), (m, n, nnz)


@pytest.mark.parametrize("s", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("nnz", [512 * 8192 - 1, 512 * 8192, 512 * 8192 + 1, 512 * 8192 + 512 * 1025, 9_000_011])
def test_plan_of_several_tiles_per_chunk(M, nnz, s):
    """Chunks of one full tile, of a tile and one sample, of a tile and a
    little more than one wavefront's part, of three tiles; one half of the
    samples in one column block."""
    m, n = 4001, 1999
    M.reset_options()
    M.set_option("balance", 0)
    M.set_option("debug", 1)
    M.init(m, n, 8, 1)
    S = samples(m, n, nnz, s, skew=True)
    order, start = oracle.block_order(S, m, n, s)
    M.plan(M.samples_to_device(S), s)
    assert np.array_equal(M.debug_plan_starts(s).cpu().numpy(), start)
    assert np.array_equal(M.debug_plan_order(nnz).cpu().numpy(), order)


def test_plan_of_more_than_32_bits_of_samples(M):
    """2^32 + 4097 samples: (block, position) rises strictly along the planned
    order and the block starts are the counts' sums, which is the stable order
    and nothing else."""
    import torch
    m, n, nnz, step = 70_001, 5003, (1 << 32) + 4097, 1 << 26
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GB of GPU memory")
    M.reset_options()
    M.set_option("balance", 0)
    M.set_option("debug", 1)
    M.init(m, n, 8, 1)
    g = torch.Generator(device="cuda").manual_seed(7)
    S = torch.zeros((nnz, 3), dtype=torch.int32, device="cuda")
    for at in range(0, nnz, step):
        b = min(step, nnz - at)
        S[at:at + b, 0] = torch.randint(0, m, (b,), device="cuda", generator=g, dtype=torch.int32)
        S[at:at + b, 1] = torch.randint(0, n, (b,), device="cuda", generator=g, dtype=torch.int32)
    S[::2, 1] = 77

    def blocks(x, s):
        return (x[:, 0].long() * s // m) * s + x[:, 1].long() * s // n

    for s in (4, 8, 16, 32, 64):
        M.plan(S, s)
        count = torch.zeros(s * s, dtype=torch.int64, device="cuda")
        for at in range(0, nnz, step):
            count += torch.bincount(blocks(S[at:at + step], s), minlength=s * s)
        start = M.debug_plan_starts(s)
        assert int(start[0]) == 0 and torch.equal(start[1:], count.cumsum(0)), s
        order = M.debug_plan_order(nnz)
        last = (-1, -1)
        for at in range(0, nnz, step):
            o = order[at:at + step]
            assert int(o.min()) >= 0 and int(o.max()) < nnz, (s, at)
            b = blocks(S[o], s)
            rises = (b[1:] > b[:-1]) | ((b[1:] == b[:-1]) & (o[1:] > o[:-1]))
            assert bool(rises.all()) and (int(b[0]), int(o[0])) > last, (s, at)
            last = int(b[-1]), int(o[-1])
        print(f"s = {s}: {nnz} samples in order", flush=True)
        del order, o, b, rises
    del S
    M.finalize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("nnz, hot, want", [(3_000_000, 0.0, 0), (3_000_000, 0.6, 1), (1 << 20, 0.0, 0),
                                            ((1 << 20) + 1, 0.6, 1), (1 << 20, 0.6, 1)])
def test_nearly_empty_blocks_do_not_switch_the_skipped_stores_on(M, nnz, hot, want):
    """All but 63 x 3 of the samples lie in the first of 64 row blocks; the
    three of every other block belong to three users.  Stores are skipped only
    where one user holds most of the first block."""
    m, n, s = 64_000, 6400, 64
    M.reset_options()
    M.init(m, n, 128, 1)
    S = samples(m, n, nnz, 3, skew=False)
    S["u"] %= m // s
    S["u"][:int(nnz * hot)] = 5
    at = np.random.default_rng(4).choice(nnz, 3 * (s - 1), replace=False)
    S["u"][at] = m // s + np.arange(3 * (s - 1)) * (m // s) // 3
    assert np.all(np.bincount(S["u"].astype(np.int64) * s // m, minlength=s)[1:] == 3)
    d = M.samples_to_device(S)
    M.plan(d, s)
    M.epoch(d, 0.0, 0.0, 0.0, "wavefront")
    assert M.get_option("blocked_skips") == want


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 255, 257, 5003])
def test_one_block_epoch_reads_the_callers_array(M, nnz, dtype):
    """Batch-Hogwild! in one XCD runs on the caller's array in place: with one
    worker it is the serial update, also of an array rewritten between two
    epochs, and with many workers every sample is used once."""
    m, n, k, lr, lam = 301, 103, 40, 0.01, 0.05
    M.reset_options()
    for key, val in dict(dtype=dtype, partition=4, workers=1).items():
        M.set_option(key, val)
    M.init(m, n, k, 3)
    P, Q = oracle.init_factors(m, n, k, 3, np.float16 if dtype else np.float32)
    d = M.samples_to_device(samples(m, n, nnz, 1, skew=False))
    for seed in (1, 2):
        S = samples(m, n, nnz, seed, skew=False)
        d.copy_(M.samples_to_device(S))
        M.epoch(d, lr, lam, lam, "hogwild")
        oracle.epoch_serial(P, Q, S, lr, lam, lam)
    tol = 2e-2 if dtype else 1e-4
    for got, want in zip(M.get_factors(m, n, k), (P, Q)):
        assert float(np.abs(got.float().cpu().numpy() - want.astype(np.float32)).max()) <= tol
    M.set_option("workers", 0)
    M.set_option("debug", 1)
    M.epoch(d, lr, lam, lam, "hogwild")
    assert bool((M.debug_visits(nnz) == 1).all())


def test_one_block_epoch_refuses_bad_indices(M):
    M.reset_options()
    M.set_option("partition", 4)
    M.init(10, 10, 8, 1)
    S = samples(10, 10, 100, 1, skew=False)
    S["v"][77] = 10
    with pytest.raises(M.MfsgdError) as e:
        M.epoch(M.samples_to_device(S), 0.01, 0.0, 0.0, "hogwild")
    assert e.value.code == M.EINVAL


@pytest.mark.parametrize("workers", [0, 1])
@pytest.mark.parametrize("k, partition, column, index", [(16, 2, 0, -1), (64, 4, 1, 97), (128, 4, 0, 1 << 30)])
def test_one_block_epoch_refuses_bad_indices_in_a_rewritten_array(M, k, partition, column, index, workers):
    """An array rewritten in place is checked again: an epoch on a bad index
    does nothing and the next call that waits says so; the call after it, and
    the next epoch, are good again."""
    import torch
    m, n, nnz = 4001, 97, 5003
    M.reset_options()
    M.set_option("partition", partition)
    M.set_option("workers", workers)
    M.init(m, n, k, 1)
    d = M.samples_to_device(samples(m, n, nnz, 1, skew=True))
    M.epoch(d, 0.01, 0.0, 0.0, "hogwild")
    assert M.get_option("hogwild_form") == 4
    before = M.get_factors(m, n, k)
    for at in (0, 2600, nnz - 1):
        good = int(d[at, column])
        d[at, column] = index
        M.epoch(d, 0.01, 0.0, 0.0, "hogwild")
        with pytest.raises(M.MfsgdError) as e:
            M.rmse(d[:0])
        assert e.value.code == M.EINVAL
        after = M.get_factors(m, n, k)
        assert torch.equal(before[0], after[0]) and torch.equal(before[1], after[1])
        d[at, column] = good
    M.epoch(d, 0.01, 0.0, 0.0, "hogwild")
    assert not torch.equal(before[0], M.get_factors(m, n, k)[0])


def test_checking_a_rewritten_array_renews_what_was_derived_from_it(M):
    """mfsgd_check_samples on a refilled buffer: the automatic form is chosen
    for the new ratings, and the forms that keep a copy train on them."""
    import torch
    m, n, k, nnz = 4000, 2000, 128, 40_000
    S = samples(m, n, nnz, 1, skew=False)
    S["u"] = S["u"] % (m // 2)  # the first half of the users
    hot = S.copy()
    hot["u"] += m // 2  # the second half, and one item with half of the samples
    hot["v"][::2] = 7
    first, second = M.samples_to_device(S), M.samples_to_device(hot)
    other = first.clone()

    def moved(P, was):  # which halves of the users the epoch updated
        d = (P != was).any(1)
        return bool(d[:m // 2].any()), bool(d[m // 2:].any())

    for opts, scheme in ((dict(partition=2), "hogwild"), (dict(partition=1), "hogwild"),
                         (dict(table_grid=16), "table"), (dict(partition=0, coherent=1, hot_log2=4), "hogwild")):
        M.reset_options()
        for key, val in opts.items():
            M.set_option(key, val)
        M.init(m, n, k, 1)
        buf = first.clone()
        keeps = opts.get("partition") == 1 or scheme == "table"

        def epoch():
            was = M.get_factors(m, n, k)[0]
            M.epoch(buf, 0.001, 0.01, 0.01, scheme)
            return moved(M.get_factors(m, n, k)[0], was)

        assert epoch() == (True, False)
        form = M.get_option("hogwild_form")
        buf.copy_(second)
        M.check_samples(other)  # another array: nothing of this one's is dropped
        assert epoch() == ((True, False) if keeps else (False, True))
        assert M.get_option("hogwild_form") == form
        M.check_samples(buf[100:101])  # a part of it
        assert epoch() == (False, True)
        if opts.get("partition") == 2:
            assert (form, M.get_option("hogwild_form")) == (0, 4)


def test_captured_one_block_epoch_keeps_its_own_length(M):
    """A captured one-XCD epoch is replayed after an epoch on a longer array:
    it trains on its own array, all of it and nothing past it."""
    import torch
    m, n, k, short, long = 301, 103, 40, 4999, 20_011
    M.reset_options()
    M.set_option("partition", 4)
    M.set_option("workers", 1)
    M.init(m, n, k, 3)
    S = samples(m, n, short, 1, skew=False)
    a, b = M.samples_to_device(S), M.samples_to_device(samples(m, n, long, 2, skew=False))
    M.epoch(a, 0.01, 0.05, 0.05, "hogwild")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        M.epoch(a, 0.01, 0.05, 0.05, "hogwild")
    P, Q = oracle.init_factors(m, n, k, 3, np.float32)
    start = [torch.from_numpy(x.copy()) for x in (P, Q)]
    oracle.epoch_serial(P, Q, S, 0.01, 0.05, 0.05)
    for _ in range(3):
        M.epoch(b, 0.01, 0.05, 0.05, "hogwild")
        M.set_factors(*start)
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip(M.get_factors(m, n, k), (P, Q)):
            assert float(np.abs(got.cpu().numpy() - want).max()) <= 1e-4


@pytest.mark.parametrize("share, form", [(1 / 60, 4), (1 / 70, 0)])
def test_automatic_form_on_large_arrays(M, share, form):
    """The largest row's share decides the automatic form (1/64); on arrays
    above 2^22 samples only rows that a subsample marks are counted in full."""
    import torch
    m, n, nnz = 300_007, 200_003, (1 << 22) + 12_345
    M.reset_options()
    M.init(m, n, 64, 1)
    g = torch.Generator(device="cuda").manual_seed(5)
    S = torch.empty((nnz, 3), dtype=torch.int32, device="cuda")
    S[:, 0] = torch.randint(0, m, (nnz,), device="cuda", generator=g, dtype=torch.int32)
    S[:, 1] = torch.randint(0, n, (nnz,), device="cuda", generator=g, dtype=torch.int32)
    S[:int(nnz * share), 1] = 123_456  # all in one place of the array
    S[:, 2] = 0
    M.epoch(S, 0.001, 0.01, 0.01, "hogwild")
    assert M.get_option("hogwild_form") == form
    S[-1, 0] = m  # one bad index anywhere is found, marked row or not
    other = S.clone()
    with pytest.raises(M.MfsgdError) as e:
        M.epoch(other, 0.001, 0.01, 0.01, "hogwild")
    assert e.value.code == M.EINVAL
