"""ckpt_solve_linear where a chain gets a wave of its own: lengths around the 64 rows a wave holds and the
limits of its launches, 32- and 64-bit arithmetic, more than 64 live entries, batches on both sides of the
rule, against the oracle; and such groups inside a ragged batch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_12499_amd import binding as B
from paper_2502_12499_amd import inputs
from test_gpu_cubic_search import one_large_size
from timing import shortest_us

pytestmark = pytest.mark.gpu


def check(d, chain_major=False):
    dc = inputs.chain_major(d)
    t = torch.from_numpy(dc if chain_major else np.ascontiguousarray(d)).cuda()
    mask, peak, status = B.ckpt_solve_linear(t, chain_major=chain_major)
    torch.cuda.synchronize()
    want_peak, want_mask = oracle.batch_solve_dynamic(dc)
    got = mask.cpu().numpy()
    assert (status.cpu().numpy() == 0).all()
    assert np.array_equal(peak.cpu().numpy(), want_peak)
    assert np.array_equal(got if chain_major else got.T, want_mask)


def live_entries(n):
    """Sizes that keep many entries of the queue alive: one large layer at the far end, tiny ones before it, so that
    the value function falls along the chain while no crossover is reached."""
    d = np.ones((n + 1, 1), dtype=np.int64)
    d[1:, 0] = np.arange(n, 0, -1)
    d[n, 0] = 1
    d[n - 1, 0] = 1 << 40
    return d


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 511, 512, 700])
def test_lengths_and_kinds_of_sizes(n):
    rng = np.random.default_rng(n)
    print(f"linear, a wave per chain: n = {n}", flush=True)
    check(inputs.uniform_aligned_chains(n, n, 9, 256, 32768), chain_major=n % 2 == 1)
    check(inputs.log_uniform_chains(n, n, 9))
    check(rng.integers(1, (1 << 62) // (n + 2), size=(n + 1, 5)).astype(np.int64))
    check(rng.integers(1, 4, size=(n + 1, 5)).astype(np.int64))
    check(np.full((n + 1, 2), 3, dtype=np.int64))
    check(np.arange(1, n + 2, dtype=np.int64)[:, None].repeat(2, 1))
    check(np.arange(n + 1, 0, -1, dtype=np.int64)[:, None].repeat(2, 1))
    check((1 << rng.integers(0, 40, size=(n + 1, 5))).astype(np.int64))
    if n > 1:
        check(live_entries(n))


@pytest.mark.parametrize("n", [7, 8, 9, 31, 32, 33, 56, 57, 72, 73, 96, 97, 160, 161])
def test_ends_of_blocks_and_limits_of_the_values(n):
    rng = np.random.default_rng(n)
    check(inputs.uniform_aligned_chains(n, n, 3, 256, 32768))
    check(inputs.log_uniform_chains(n, n, 3))
    for most in (1 << 30, 1 << 62, (1 << 63) - 1):  # of sum(d) + max(d): 32 bits, 64 bits, what only the list takes
        for at in (0, n // 2, n):
            d = np.stack([rng.integers(1, max(2, most // (4 * n)), size=n + 1) for _ in range(3)], axis=1).astype(np.int64)
            d[(at + 1) % (n + 1)] |= 1
            for c in range(3):  # the size at `at` takes sum(d) + max(d) about to `most`, and not beyond INT64_MAX
                rest = int(d[:, c].sum()) - int(d[at, c])
                d[at, c] = (most - 1 + c - rest) // 2 if most < (1 << 63) - 1 else (most - c - rest) // 2
                assert rest + 2 * int(d[at, c]) <= (1 << 63) - 1
            check(d)


@pytest.mark.parametrize("n, batch", [(3, 60), (16, 1100), (17, 60), (63, 60), (64, 1100), (64, 65600), (65, 1100), (100, 60), (300, 1100)])
def test_the_upper_half_of_32_bits(n, batch):
    """sum(d) + max(d) between 2**31 and 2**32, and on both sides of 2**32 - 2, from where on values are wider: a wave per
    chain, rows, and rows of what the lanes leave."""
    rng = np.random.default_rng(n * batch)
    d = rng.integers((1 << 31) // (n + 1), (1 << 32) // (n + 2), size=(n + 1, batch)).astype(np.int64)
    for c in range(0, batch, 3):
        at, most = int(rng.integers(0, n + 1)), (1 << 32) - int(rng.integers(0, 6))
        if c % 2:  # one size is half of it
            d[:, c] = rng.integers(1, max(2, most // (4 * n)), size=n + 1)
        d[at, c] = 0
        d[at, c] = (most - int(d[:, c].sum())) // 2
        if 2 * int(d[at, c]) + int(d[:, c].sum()) - int(d[at, c]) < most:
            d[(at + 1) % (n + 1), c] += 1
    assert d.min() > 0
    print(f"linear, upper half of 32 bits: n = {n}, batch = {batch}", flush=True)
    check(d, chain_major=n % 2 == 1)


@pytest.mark.parametrize("n", [2047, 2048, 3000])
def test_long_chains(n):
    check(inputs.uniform_aligned_chains(n, n, 2, 256, 32768))
    check(live_entries(n))


@pytest.mark.parametrize("n, batch", [(2047, 512), (2047, 513), (1279, 1024), (1280, 1024), (2048, 4)])
def test_a_list_of_their_own_where_all_waves_fit_the_chip(n, batch):
    d = inputs.uniform_aligned_chains(4, n, batch, 256, 32768)
    d[:, 1:3] = live_entries(n)                                                  # more than 64 live entries: for the list
    d[:, batch - 1] = live_entries(n)[:, 0]
    check(d)


@pytest.mark.parametrize("batch", [1024, 1025, 65536, 65537])
def test_batches_on_both_sides_of_the_rule(batch):
    d = inputs.uniform_aligned_chains(3, 40, batch, 256, 32768)
    d[:, ::9] += 1
    check(d)


def test_bad_chains_are_reported_alone():
    for n in (100, 600):
        d = inputs.uniform_aligned_chains(4, n, 12, 256, 32768)
        want_peak, want_mask = oracle.batch_solve_dynamic(inputs.chain_major(d))
        d[n, 2] = 0
        d[:, 7] = (1 << 62) + 3
        d[0, 11] = -4
        mask, peak, status = B.ckpt_solve_linear(torch.from_numpy(d).cuda())
        torch.cuda.synchronize()
        ok = np.array([c for c in range(12) if c not in (2, 7, 11)])
        st = status.cpu().numpy()
        assert (st[ok] == 0).all() and st[[2, 7, 11]].tolist() == [3, 4, 3]
        assert (peak.cpu().numpy()[[2, 7, 11]] == -1).all() and not mask.cpu().numpy()[:, [2, 7, 11]].any()
        assert np.array_equal(peak.cpu().numpy()[ok], want_peak[ok])
        assert np.array_equal(mask.cpu().numpy().T[ok], want_mask[ok])


def check_one_large_size(results, d, fits):
    """d: chains of equal length, the first sixteen of them over and over."""
    mask, peak, status = results
    good = np.ascontiguousarray(np.where(fits[None, :], d, 1)[:, :16])
    want_peak, want_mask = oracle.batch_solve_dynamic(inputs.chain_major(good))
    assert status.tolist() == [0 if f else 4 for f in fits]
    for c in range(d.shape[1]):
        if fits[c]:
            assert peak[c] == want_peak[c % 16] and np.array_equal(mask[:, c], want_mask[c % 16])
        else:
            assert peak[c] == -1 and not mask[:, c].any()


@pytest.mark.parametrize("n", [2, 3, 64, 200, 511, 512, 700])
def test_one_size_near_the_largest_value(n):
    """sum(d) + max(d) wraps around 2^64 for some of these chains."""
    d, fits = one_large_size(n)
    print(f"linear, one large size: n = {n}", flush=True)
    check_one_large_size([t.cpu().numpy() for t in B.ckpt_solve_linear(torch.from_numpy(d).cuda())], d, fits)


@pytest.mark.parametrize("n,batch", [(3, 65552), (64, 65552), (65, 65552), (300, 65552), (20000, 16)])
def test_one_size_near_the_largest_value_a_lane_per_chain(n, batch):
    d, fits = one_large_size(n)
    d, fits = np.tile(d, (1, batch // 16)), np.tile(fits, batch // 16)
    print(f"linear, one large size: n = {n}, batch = {batch}", flush=True)
    check_one_large_size([t.cpu().numpy() for t in B.ckpt_solve_linear(torch.from_numpy(d).cuda())], d, fits)


def test_one_size_near_the_largest_value_in_a_ragged_batch():
    d, fits = one_large_size(300)
    flat = torch.from_numpy(np.ascontiguousarray(d.T).reshape(-1)).cuda()
    off = np.arange(17, dtype=np.int64) * 301
    mask, peak, status = (t.cpu().numpy() for t in B.ckpt_ragged_solve_linear(flat, off))
    check_one_large_size((mask.reshape(16, 301).T, peak, status), d, fits)


@pytest.mark.parametrize("short", [0, 262144])
def test_long_groups_of_a_ragged_batch(short):
    """Staged (beside `short` chains of one layer), groups on both sides of the rule (257 and 4095 layers get waves, 256 and
    4096 lanes), with chains that leave either kind; the same chains without the others, which are taken where they lie.
    Lengths counted on the host and on the device."""
    rng = np.random.default_rng(1)
    lengths = np.concatenate([np.array([256, 257, 257, 1001, 4095, 4096, 300, 300, 300]),
                              rng.choice([5, 24, 300], size=200), np.ones(short, dtype=np.int64)])
    rng.shuffle(lengths)
    d, _, off = inputs.ragged_batch(6, lengths)
    for c in range(0, len(lengths), 3 if short == 0 else 1000):
        d[off[c]:off[c + 1]] += 1
    for c in np.nonzero(lengths == 300)[0][3:50:3]:
        d[off[c]:off[c + 1]] += 1
    for c in np.nonzero(lengths == 300)[0][:3]:
        d[off[c]:off[c + 1]] = live_entries(300)[:, 0]
    want_peak, want_mask = oracle.ragged_solve_dynamic(d, off)
    for off_dev in (None, torch.from_numpy(off).cuda()):
        mask, peak, status = B.ckpt_ragged_solve_linear(torch.from_numpy(d).cuda(), off, offsets_dev=off_dev)
        torch.cuda.synchronize()
        assert (status.cpu().numpy() == 0).all()
        assert np.array_equal(peak.cpu().numpy(), want_peak)
        assert np.array_equal(mask.cpu().numpy(), want_mask)


@pytest.mark.parametrize("batch, short", [(3000, 0), (12288, 0), (3000, 262144), (12288, 262144)])
def test_many_long_chains_of_a_ragged_batch(batch, short):
    """Groups of 257 to 300 layers and some of 40, taken where they lie, and staged beside `short` chains of one layer: a
    wave to a chain, and (all of them together being too many) a lane."""
    rng = np.random.default_rng(batch)
    lengths = np.where(rng.random(batch) < 0.1, 40, rng.integers(257, 301, size=batch))
    lengths = np.concatenate([lengths, np.ones(short, dtype=np.int64)])
    d, _, off = inputs.ragged_batch(8, lengths)
    for c in range(0, batch, 5):
        d[off[c]:off[c + 1]] += 1
    want_peak, want_mask = oracle.ragged_solve_dynamic(d, off)
    for off_dev in (None, torch.from_numpy(off).cuda()):
        mask, peak, status = B.ckpt_ragged_solve_linear(torch.from_numpy(d).cuda(), off, offsets_dev=off_dev)
        torch.cuda.synchronize()
        assert (status.cpu().numpy() == 0).all()
        assert np.array_equal(peak.cpu().numpy(), want_peak)
        assert np.array_equal(mask.cpu().numpy(), want_mask)


# sum(d) + max(d) up to 2^61, which signed 64-bit values of the recurrence have room for, and beyond 2^62
@pytest.mark.parametrize("least, most", [(0, 61), (62, 63)])
@pytest.mark.parametrize("batch, n", [(1, 152), (1000, 64), (2048, 64), (16384, 64), (65536, 12), (65536, 64), (65537, 64),
                                      (131072, 17)])
def test_what_64_bits_cost(batch, n, least, most):
    """Chains that need 64 bits go with the others' kernels, in wider arithmetic, and not one after the other to a lane or
    a wave: four to twenty times as long then, up to 2.4 times so."""
    rng = np.random.default_rng(n)
    aligned = torch.from_numpy(inputs.uniform_aligned_chains(1, n, batch, 256, 32768)).cuda()
    lo = (1 << least) // (n + 2) + 1
    wide = torch.from_numpy(rng.integers(lo, ((1 << most) - 1) // (n + 2), size=(n + 1, batch)).astype(np.int64) | 1).cuda()
    a, w = (shortest_us(lambda: B.ckpt_solve_linear(d)) for d in (aligned, wide))
    print(f"{batch} chains of {n} layers: aligned {a:.1f} us, in 64 bits {w:.1f} us", flush=True)
    assert w < 4 * a


def test_what_two_kinds_of_deferred_chains_cost():
    """Deferred chains with and without large sizes, side by side in every wave, cost what one kind does: 1.7 times that
    with a list's end and an atomic for each, 1.0 with one atomic a wave."""
    lo = torch.randint(1 << 40, 1 << 43, (5, 1048576), device="cuda") * 2 + 1
    mixed = lo.clone()
    mixed[2, ::2] += 1 << 45
    one, two = (shortest_us(lambda: B.ckpt_solve_linear(d)) for d in (lo, mixed))
    print(f"1,048,576 chains of 4 layers: {one:.1f} us, with large ones among them {two:.1f} us", flush=True)
    assert two < 1.3 * one
