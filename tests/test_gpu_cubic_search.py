"""ckpt_solve_cubic on the lengths and sizes where its search over the budgets changes form, against the
oracle: blocks of eight positions, slices of 64, 32- and 64-bit arithmetic, prefix sums beyond 32 bits,
repeated budgets, ties, batches on both sides of the split into two launches."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_12499_amd import binding as B
from paper_2502_12499_amd import inputs
from timing import shortest_us

pytestmark = pytest.mark.gpu


def check(d, chain_major=False):
    dc = inputs.chain_major(d)
    t = torch.from_numpy(dc if chain_major else np.ascontiguousarray(d)).cuda()
    mask, peak, budget, status = B.ckpt_solve_cubic(t, chain_major=chain_major)
    torch.cuda.synchronize()
    want_peak, want_mask, want_s = oracle.batch_solve_static(dc)
    got = mask.cpu().numpy()
    assert (status.cpu().numpy() == 0).all()
    assert np.array_equal(peak.cpu().numpy(), want_peak)
    assert np.array_equal(budget.cpu().numpy(), want_s)
    assert np.array_equal(got if chain_major else got.T, want_mask)


@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 16, 63, 64, 65, 127, 128, 129, 255, 256])
def test_lengths_and_kinds_of_sizes(n):
    rng = np.random.default_rng(n)
    b = 24 if n <= 65 else 4
    print(f"cubic search: n = {n}", flush=True)
    check(inputs.uniform_aligned_chains(n, n, b, 256, 32768), chain_major=n % 2 == 1)
    check(inputs.log_uniform_chains(n, n, b))                                    # sums beyond 32 bits
    check(rng.integers(1, (1 << 62) // (n + 2), size=(n + 1, b)).astype(np.int64))  # 64-bit arithmetic
    check(rng.integers(1, 4, size=(n + 1, b)).astype(np.int64))                  # ties, few values
    check((1 << rng.integers(0, 40, size=(n + 1, b))).astype(np.int64))          # one layer outweighs the rest
    check(np.arange(1, n + 2, dtype=np.int64)[:, None].repeat(2, 1))
    alternating = np.ones((n + 1, 2), dtype=np.int64)
    alternating[::2, 0] = 1000003
    alternating[1::2, 1] = 999999937
    check(alternating)


@pytest.mark.parametrize("batch", [1023, 1024, 1600])
def test_batches_on_both_sides_of_the_split(batch):
    d = inputs.uniform_aligned_chains(3, 20, batch, 256, 32768)
    wide = np.random.default_rng(batch).integers(1, 1 << 50, size=(21, batch)).astype(np.int64)
    d[:, ::7] = wide[:, ::7]                                                     # every seventh needs 64 bits
    check(d)


@pytest.mark.parametrize("n,batch", [(1, 8192), (2, 8193), (5, 16385), (36, 16391), (37, 8199), (63, 16384), (64, 8195), (72, 16387),
                                     (73, 16386), (96, 8197), (97, 4099), (120, 4096), (128, 8198), (129, 2048), (200, 2051), (256, 2063)])
def test_rows_of_lanes(n, batch):
    """Batches whose chains have rows of 8 or 16 lanes each: lengths around a block, a ring and the lanes' shares; a wave's
    chains of every kind side by side, chains that are left to a wave each and bad ones among them."""
    rng = np.random.default_rng(n)
    print(f"rows of lanes: n = {n}, batch = {batch}", flush=True)
    kinds = [inputs.uniform_aligned_chains(n, n, 61, 256, 32768), inputs.log_uniform_chains(n, n, 61),
             np.stack([network(n, k)[:, 0] if n > 4 else np.full(n + 1, k + 1) for k in range(61)], 1),
             rng.integers(1 << 24, 1 << 26, size=(n + 1, 19)), rng.integers(1, 4, size=(n + 1, 7)),
             np.full((n + 1, 1), 7), rng.integers(1, (1 << 62) // (n + 2), size=(n + 1, 3)),
             (1 << rng.integers(0, 40, size=(n + 1, 5)))]
    d = np.concatenate([k.astype(np.int64) for k in kinds], axis=1)
    d = d[:, rng.permutation(d.shape[1])]
    some = d.shape[1]
    want_peak, want_mask, want_s = oracle.batch_solve_static(inputs.chain_major(d))
    at = np.arange(batch) % some
    d = d[:, at]
    d[n // 2, 7::1009] = 0
    bad = d.min(0) <= 0
    mask, peak, budget, status = B.ckpt_solve_cubic(torch.from_numpy(np.ascontiguousarray(d)).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(status.cpu().numpy(), np.where(bad, 3, 0))
    assert np.array_equal(peak.cpu().numpy(), np.where(bad, -1, want_peak[at]))
    assert np.array_equal(budget.cpu().numpy(), np.where(bad, -1, want_s[at]))
    assert np.array_equal(mask.cpu().numpy().T, np.where(bad[:, None], 0, want_mask[at]))


def front_heavy(n, seed, batch):
    """Layers in front that outweigh the rest: sizes that fall from layer to layer, pictures halved in the first third, a few
    large layers before many small ones."""
    rng = np.random.default_rng(seed)
    k = np.arange(n + 1)[:, None]
    falls = 2.0 ** 27 * (0.8 + 0.15 * rng.random(batch)) ** k * (0.7 + 0.6 * rng.random((n + 1, batch)))
    ends = np.sort(1 + rng.random((4, batch)) * n / 3, axis=0)
    halved = (k[:, :, None] >= ends.T[None]).sum(2)
    pyramid = rng.integers(8, 208, size=batch) * 802816.0 / 2.0 ** halved
    small = np.where(k < 5, rng.integers(1 << 20, 1 << 21, size=(n + 1, batch)), rng.integers(1024, 5120, size=(n + 1, batch)))
    at = np.arange(batch) % 3
    return np.maximum(np.where(at == 0, falls, np.where(at == 1, pyramid, small)).astype(np.int64), 1)


@pytest.mark.parametrize("share", ["all", "tenth", "half in front"])
@pytest.mark.parametrize("n,batch", [(44, 8192), (64, 8197), (72, 16390), (100, 4099), (152, 2051), (152, 9001), (256, 2048)])
def test_windows_beyond_the_ring(n, batch, share):
    """Chains that the rows leave to waves: of the whole batch, of some, side by side with others or not; bad ones and ones that
    need 64 bits among them."""
    print(f"windows beyond the ring: n = {n}, batch = {batch}, {share}", flush=True)
    rng = np.random.default_rng(n + batch)
    far, near = front_heavy(n, n, 30), inputs.log_uniform_chains(n, n, 29)
    wide = rng.integers(1, (1 << 62) // (n + 2), size=(n + 1, 2))
    kinds = np.concatenate([far, near, wide], axis=1).astype(np.int64)
    want_peak, want_mask, want_s = oracle.batch_solve_static(inputs.chain_major(kinds))
    c = np.arange(batch)
    is_far = {"all": c >= 0, "tenth": c % 10 == 3, "half in front": c < batch // 2}[share]
    at = np.where(is_far, c % 30, 30 + c % 29)
    at[5::997] = 59 + c[5::997] % 2
    d = kinds[:, at]
    d[n // 2, 7::1009] = 0
    bad = d.min(0) <= 0
    major = n in (44, 100)
    mask, peak, budget, status = B.ckpt_solve_cubic(torch.from_numpy(np.ascontiguousarray(d.T if major else d)).cuda(), chain_major=major)
    torch.cuda.synchronize()
    assert np.array_equal(status.cpu().numpy(), np.where(bad, 3, 0))
    assert np.array_equal(peak.cpu().numpy(), np.where(bad, -1, want_peak[at]))
    assert np.array_equal(budget.cpu().numpy(), np.where(bad, -1, want_s[at]))
    assert np.array_equal(mask.cpu().numpy() if major else mask.cpu().numpy().T, np.where(bad[:, None], 0, want_mask[at]))


@pytest.mark.parametrize("n,batch", [(3, 8192), (16, 8195), (33, 16384), (64, 16390), (100, 4096), (200, 2049)])
def test_rows_with_one_large_size(n, batch):
    """One size of which five add up to about 2^32, in front, inside or last, others whose sums stay below that or do not."""
    print(f"rows with one large size: n = {n}, batch = {batch}", flush=True)
    rng = np.random.default_rng(n)
    d = np.concatenate([rng.integers(1, 1 << b, size=(n + 1, 20)) for b in (12, 20, 26)], axis=1) | 1
    d[rng.integers(0, n + 1, size=60), np.arange(60)] = rng.integers(600_000_000, 860_000_000, size=60)
    d = d.astype(np.int64)
    want_peak, want_mask, want_s = oracle.batch_solve_static(inputs.chain_major(d))
    at = rng.integers(0, 60, size=batch)
    mask, peak, budget, status = B.ckpt_solve_cubic(torch.from_numpy(np.ascontiguousarray(d[:, at])).cuda())
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    assert np.array_equal(peak.cpu().numpy(), want_peak[at])
    assert np.array_equal(budget.cpu().numpy(), want_s[at])
    assert np.array_equal(mask.cpu().numpy().T, want_mask[at])


@pytest.mark.parametrize("n", [152, 256])
def test_windows_beyond_the_ring_take_no_longer_than_a_wave_a_chain(n):
    """2,047 chains have a wave each, twice as many would have rows: with the rows' rounds before them and in the arithmetic of
    64 bits they took 5.7 and 5.8 times as long, not 1.7 and 1.8 times."""
    d = np.tile(front_heavy(n, n, 89), 46)[:, :4094]
    once, twice = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (d[:, :2047], d))
    ws = torch.empty(B.workspace_bytes(B.CALL_SOLVE_CUBIC, B.layout_of(twice)), dtype=torch.uint8, device="cuda")
    few, many = (shortest_us(lambda: B.ckpt_solve_cubic(x, workspace=ws)) for x in (once, twice))
    print(f"{few:.0f} and {many:.0f} us", flush=True)
    assert many < 2.6 * few


def test_bad_chains_are_reported_alone():
    d = inputs.uniform_aligned_chains(4, 30, 1100, 256, 32768)
    dc = inputs.chain_major(d)
    want_peak, want_mask, want_s = oracle.batch_solve_static(dc)
    d[5, 3] = 0
    d[:, 700] = (1 << 62) + 1
    d[30, 1099] = -1
    for batch in (800, 1100):
        mask, peak, budget, status = B.ckpt_solve_cubic(torch.from_numpy(np.ascontiguousarray(d[:, :batch])).cuda())
        torch.cuda.synchronize()
        bad = np.array([c for c in (3, 700, 1099) if c < batch])
        ok = np.setdiff1d(np.arange(batch), bad)
        st = status.cpu().numpy()
        assert (st[ok] == 0).all() and st[bad].tolist() == [3, 4, 3][:len(bad)]
        assert (peak.cpu().numpy()[bad] == -1).all() and (budget.cpu().numpy()[bad] == -1).all()
        assert not mask.cpu().numpy()[:, bad].any()
        assert np.array_equal(peak.cpu().numpy()[ok], want_peak[ok])
        assert np.array_equal(budget.cpu().numpy()[ok], want_s[ok])
        assert np.array_equal(mask.cpu().numpy().T[ok], want_mask[ok])


def one_large_size(n):
    """Chains (n+1, 16) of small sizes with one near the largest 64-bit value, and whether sum(d) + max(d) still fits:
    the large size in front, inside and at the end; up to half of the largest value it does."""
    top = (1 << 63) - 1
    columns = []
    for k in (0, 1, n // 2, n):
        for large in (top, top - (1 << 31), (top - n) // 2 + 1, (top - n) // 2):
            x = np.ones(n + 1, dtype=np.int64)
            x[k] = large
            columns.append(x)
    d = np.stack(columns, axis=1)
    fits = [sum(map(int, x)) + int(x.max()) <= top for x in columns]
    assert fits.count(True) == 4
    return d, np.array(fits)


@pytest.mark.parametrize("n", [2, 3, 64, 142, 200, 257, 300])
@pytest.mark.parametrize("batch", [16, 1040])
def test_one_size_near_the_largest_value(n, batch):
    """sum(d) + max(d) wraps around 2^64 for some of these chains."""
    if batch > 16 and n > 64:
        batch = 528                                                              # (a lane per point up to 256 layers)
    d, fits = one_large_size(n)
    d = np.tile(d, (1, batch // 16))
    fits = np.tile(fits, batch // 16)
    print(f"one large size: n = {n}, batch = {batch}", flush=True)
    good = np.where(fits[None, :], d, 1)
    want_peak, want_mask, want_s = oracle.batch_solve_static(inputs.chain_major(np.ascontiguousarray(good[:, :16])))
    mask, peak, budget, status = (t.cpu().numpy() for t in B.ckpt_solve_cubic(torch.from_numpy(d).cuda()))
    assert status.tolist() == [0 if f else 4 for f in fits]
    for c in range(batch):
        if fits[c]:
            assert peak[c] == want_peak[c % 16] and budget[c] == want_s[c % 16]
            assert np.array_equal(mask[:, c], want_mask[c % 16])
        else:
            assert peak[c] == -1 and budget[c] == -1 and not mask[:, c].any()


@pytest.mark.parametrize("batch,offsets_on_device", [(300, False), (1500, True)])
def test_ragged_batches_of_short_chains(batch, offsets_on_device):
    """Every class of lengths, both arithmetics, a bad chain among them."""
    rng = np.random.default_rng(batch)
    lengths = np.concatenate([np.array([1, 2, 32, 33, 64, 65, 128, 129, 256]), rng.integers(1, 40, size=batch - 9)])
    rng.shuffle(lengths)
    d, _, off = inputs.ragged_batch(batch, lengths)
    for c in range(0, batch, 5):                                                 # 64-bit arithmetic
        d[off[c]:off[c + 1]] = rng.integers(1, 1 << 52, size=off[c + 1] - off[c])
    want_peak, want_mask, want_s = oracle.ragged_solve_static(d, off)
    bad = batch // 2
    d[off[bad]] = -5
    t = torch.from_numpy(d).cuda()
    mask, peak, budget, status = B.ckpt_ragged_solve_cubic(
        t, off, offsets_dev=torch.from_numpy(off).cuda() if offsets_on_device else None)
    torch.cuda.synchronize()
    ok = np.arange(batch) != bad
    st = status.cpu().numpy()
    assert (st[ok] == 0).all() and st[bad] == 3
    assert np.array_equal(peak.cpu().numpy()[ok], want_peak[ok]) and peak.cpu().numpy()[bad] == -1
    assert np.array_equal(budget.cpu().numpy()[ok], want_s[ok]) and budget.cpu().numpy()[bad] == -1
    got = mask.cpu().numpy()
    keep = np.ones(len(d), dtype=bool)
    keep[off[bad]:off[bad + 1]] = False
    assert np.array_equal(got[keep], want_mask[keep]) and not got[~keep].any()


def network(n, seed):
    """Layer sizes of a bottleneck network: every size a multiple of the batch size, many sums repeated."""
    rng = np.random.default_rng(seed)
    batch, width, pixels = int(rng.integers(9, 250)), 16 * int(rng.integers(1, 5)), 8 * int(rng.integers(7, 29))
    ends = np.sort(rng.integers(2, n, size=3))
    sizes = [batch * 12 * (2 * pixels) ** 2, batch * 4 * width * pixels ** 2]
    for k in range(2, n):
        stage = int(np.searchsorted(ends, k, side="right"))
        w, hw = width << stage, max(pixels >> stage, 1)
        sizes.append(batch * 4 * (4 * w if k % 3 == 1 else w) * hw * hw)
    sizes.append(batch * 4000)
    return np.array(sizes, dtype=np.int64)[:, None]


@pytest.mark.parametrize("n", [257, 319, 320, 321, 511, 512, 640])
def test_long_chains(n):
    """One wave per point: slices of 64 positions, windows that reach back beyond two of them, the
    greatest common divisor, 32- and 64-bit values."""
    rng = np.random.default_rng(n)
    print(f"cubic search, long chains: n = {n}", flush=True)
    check(inputs.uniform_aligned_chains(n, n, 3, 256, 32768), chain_major=n % 2 == 1)
    check(inputs.log_uniform_chains(n, n, 2))
    check(network(n, n))
    check(rng.integers(1, (1 << 62) // (n + 2), size=(n + 1, 1)).astype(np.int64))
    check(rng.integers(1, 4, size=(n + 1, 2)).astype(np.int64))
    check(np.full((n + 1, 1), 3 << 40, dtype=np.int64))
    check((1 << rng.integers(0, 40, size=(n + 1, 1))).astype(np.int64))
    check(np.arange(n + 1, 0, -1, dtype=np.int64)[:, None].copy())
    heavy_ends = np.ones((n + 1, 1), dtype=np.int64)                             # one window over hundreds of layers
    heavy_ends[n // 2] = 1 << 30
    check(heavy_ends)


@pytest.mark.parametrize("n", [191, 192, 193, 959, 960, 1023, 1024, 1025, 1087, 1088])
def test_the_last_wave_of_the_table_that_holds_sizes(n):
    """The waves and threads that a chain's sizes end in: its last size alone there, a common divisor of all sizes that it
    alone takes away, 64-bit arithmetic, and a chain whose last size alone is bad."""
    rng = np.random.default_rng(n)
    d = rng.integers(1, 1000, size=(n + 1, 4)).astype(np.int64)
    d[:, 1] *= 3 * (1 << 30) + 9                    # 32 bits once divided
    d[:, 2] *= 3 * (1 << 30) + 9
    d[n, 2] += 1                                    # not so
    d[n, 3] = 1 << 40
    print(f"cubic search, table: n = {n}", flush=True)
    check(d, chain_major=n % 2 == 1)
    d[n, 1], d[n, 3] = 0, -(1 << 40)
    status = B.ckpt_solve_cubic(torch.from_numpy(d).cuda())[3].cpu().tolist()
    assert [s == 0 for s in status] == [True, False, True, False]


@pytest.mark.parametrize("n", [64, 142, 200, 257, 300, 640])
def test_sizes_at_the_ends_that_outweigh_the_rest(n):
    """The size in front, or the last one, 2^20 to 2^50 times the interior sizes: neither is part of any budget."""
    rng = np.random.default_rng(n)
    columns = []
    for k in (0, n):
        for shift in (24, 34, 40, 43, 50, 61):
            for kind in range(3):
                x = [np.full(n + 1, 100), rng.integers(1, 1000001, size=n + 1), rng.integers(1, 4, size=n + 1)][kind]
                x = x.astype(np.int64)
                x[k] = 1 << shift
                columns.append(x)
    d = np.stack(columns, axis=1)
    check(d)
    for c in (6, 7, 24):                                                         # one chain: more points to a round
        check(d[:, c:c + 1])


@pytest.mark.parametrize("n", [2, 3, 8, 24, 64, 100, 129, 142, 200, 300, 640])
def test_layers_that_outweigh_the_rest(n):
    """Sizes of very different orders: two rounds of evenly placed points leave most budgets in one interval."""
    rng = np.random.default_rng(n)
    plain = rng.integers(1, 1000001, size=n + 1).astype(np.int64)
    columns = []
    for at, size in (((1,), 10**9), ((n // 3,), 10**14), ((n - 1,), 10**15), ((n // 2,), 10**18),
                     ((n // 4, n // 2), 10**15), ((n // 5, n // 4, n // 3, n // 2), 10**16)):
        x = plain.copy()
        for k, place in enumerate(at):
            x[place] = size + 12345 * k if len(at) == 2 else size // 1000**k
        columns.append(x)
    columns.append(1 << rng.integers(0, 50, size=n + 1))
    columns.append(np.exp2(45 * rng.random(n + 1)).astype(np.int64) + 1)
    columns.append(np.where(np.arange(n + 1) % 2 == 0, 1000003, 999999937))
    d = np.stack(columns, axis=1).astype(np.int64)
    print(f"cubic search, sizes of different orders: n = {n}", flush=True)
    check(d)                                                                     # few waves to a chain
    check(np.tile(d, (1, 120 if n <= 128 else 60)) if n < 300 else d[:, ::-1])   # the other form, or its other launch
    for c in (1, 2, 3, 4, 5, 7):
        check(d[:, c:c + 1])                                                     # many


def test_a_chain_whose_budgets_several_workgroups_list():
    rng = np.random.default_rng(1100)
    plain = rng.integers(1, 1000001, size=1101).astype(np.int64)
    heavy = plain.copy()
    heavy[366] = 10**15
    print("cubic search: 1,100 layers, one of 10^15", flush=True)
    check(heavy[:, None])
    heavy[800] = 10**15 + 12345
    check(np.stack([plain, heavy], axis=1))


@pytest.mark.parametrize("batch", [2, 33])
def test_batches_of_long_chains(batch):
    d = inputs.uniform_aligned_chains(7, 270, batch, 256, 32768)
    d[:, 1] = inputs.log_uniform_chains(8, 270, 1)[:, 0]
    want_peak, want_mask, want_s = oracle.batch_solve_static(inputs.chain_major(d))
    if batch > 2:
        d[100, 5] = 0
    mask, peak, budget, status = B.ckpt_solve_cubic(torch.from_numpy(np.ascontiguousarray(d)).cuda())
    torch.cuda.synchronize()
    ok = np.arange(batch) != 5
    assert status.cpu().numpy().tolist() == [0 if k else 3 for k in ok]
    assert np.array_equal(peak.cpu().numpy()[ok], want_peak[ok])
    assert np.array_equal(budget.cpu().numpy()[ok], want_s[ok])
    assert np.array_equal(mask.cpu().numpy().T[ok], want_mask[ok])
    if batch > 2:
        assert peak[5] == -1 and budget[5] == -1 and not mask[:, 5].any()



# Up to 256 layers a wave takes a point in batches of up to 512 chains of more than 128 layers where the workspace has
# the room (from 128 to 141 layers on), else a lane does: both forms at the same lengths.
@pytest.mark.parametrize("n", [128, 129, 136, 141, 142, 200, 255, 256])
def test_both_forms_of_the_search(n):
    for batch in (1, 2, 8):
        check(inputs.uniform_aligned_chains(n, n, batch, 256, 32768))
        check(inputs.log_uniform_chains(n + 1, n, batch), chain_major=True)


@pytest.mark.parametrize("batch", [512, 513])
def test_both_forms_around_the_largest_batch(batch):
    check(inputs.uniform_aligned_chains(5, 150, batch, 1, 4))


@pytest.mark.parametrize("n", [130, 256, 257, 320, 1001])
def test_repeated_layers(n):
    """Equal values among which the passes take the last predecessor and the canonical set the first: next to each other,
    a slice apart, and farther back than the slices in registers."""
    k = np.arange(n + 1)
    chains = [np.full(n + 1, 5), np.where(k % 3 == 2, 16, 4), np.where(k % 97 == 40, 1, 1000), np.where(k % 150 == 20, 7, 100 + k % 5),
              1 + k % 2]
    print(f"repeated layers: n = {n}", flush=True)
    check(np.stack(chains, axis=1).astype(np.int64))
    check((np.stack(chains[1:3], axis=1).astype(np.int64)) * ((1 << 40) + 1))     # the same in 64 bits


def test_what_the_budgets_of_several_chains_cost():
    """The budgets that a round of points leaves of several chains are cut by a second round where they are many: finishing
    them took 16 unrounded chains of 129 and 200 layers 1.9 to 2.4 times what one takes, 1.2 to 1.4 so."""
    for n in (129, 200):
        for seed in range(3):
            d = torch.from_numpy(inputs.log_uniform_chains(seed, n, 16)).cuda()
            one = shortest_us(lambda: B.ckpt_solve_cubic(d[:, :1].contiguous()))
            many = shortest_us(lambda: B.ckpt_solve_cubic(d))
            print(f"{n} unrounded layers: one chain {one:.1f} us, 16 {many:.1f} us", flush=True)
            assert many < 1.75 * one


def test_what_a_few_long_chains_of_a_ragged_batch_cost():
    """Sixteen long chains that need 64 bits among a thousand short ones cost what they cost alone, not twice that."""
    rng = np.random.default_rng(2)
    lengths = np.full(1023, 24)
    lengths[rng.permutation(1023)[:16]] = 256

    def us(lengths):
        off = np.zeros(len(lengths) + 1, dtype=np.int64)
        np.cumsum(lengths + 1, out=off[1:])
        d = torch.from_numpy(np.floor(2 ** rng.uniform(16, 28, size=off[-1])).astype(np.int64)).cuda()
        return shortest_us(lambda: B.ckpt_ragged_solve_cubic(d, off))

    together, alone = us(lengths), us(lengths[lengths == 256])
    print(f"16 unrounded chains of 256 layers {alone:.1f} us, with 1,007 of 24 {together:.1f} us", flush=True)
    assert together < 1.5 * alone
