"""ckpt_solve_linear where four chains share a wave: lengths around the 16 positions of a block, 32-bit integers, doubles and
chains that need more, queues that outgrow a row, batches on both sides of the rules, against the oracle; and the same in
ragged calls, whose chains are taken where they lie."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_12499_amd import binding as B
from paper_2502_12499_amd import inputs
from test_gpu_linear_wave import check, live_entries

pytestmark = pytest.mark.gpu
MORE_THAN_WAVES = 1025  # chains: four to a wave


def kinds(n, batch, seed):
    """Chains of every kind side by side, so that a wave's rows differ: aligned, unrounded (doubles), up to 2^52 and
    beyond, small, equal, ascending, powers of two, many live entries."""
    rng = np.random.default_rng(seed)
    d = np.empty((n + 1, batch), dtype=np.int64)
    for c in range(batch):
        k = c % 11
        if k == 0:
            d[:, c] = 4096 * rng.integers(256, 32769, size=n + 1)
        elif k == 1:
            d[:, c] = np.floor(2 ** rng.uniform(16, 28, size=n + 1))
        elif k == 2:
            d[:, c] = rng.integers(1, (1 << 52) // (n + 2), size=n + 1)
        elif k == 3:
            d[:, c] = rng.integers(1, (1 << 62) // (n + 2), size=n + 1)
        elif k == 4:
            d[:, c] = rng.integers(1, 4, size=n + 1)
        elif k == 5:
            d[:, c] = 3
        elif k == 6:
            d[:, c] = np.arange(1, n + 2) * (1 + c % 7)
        elif k == 7:
            d[:, c] = np.arange(n + 1, 0, -1)
        elif k == 8:
            d[:, c] = 1 << rng.integers(0, 40, size=n + 1)
        elif k == 9:
            d[:, c] = live_entries(n)[:, 0] if n > 1 else 5
        else:
            d[:, c] = 4096 * rng.integers(256, 32769, size=n + 1)
    return d


@pytest.mark.parametrize("n", [1, 2, 7, 15, 16, 17, 31, 32, 33, 47, 48, 63, 64, 65, 152, 320, 321])
def test_lengths_and_kinds_of_sizes(n):
    print(f"linear, four chains a wave: n = {n}", flush=True)
    check(kinds(n, MORE_THAN_WAVES + 3 * 11, n), chain_major=n % 2 == 1)


@pytest.mark.parametrize("n, unrounded", [(16, 3000), (17, 900), (17, 65600), (33, 3000), (130, 900), (130, 3000)])
def test_what_the_lanes_of_a_larger_batch_leave(n, unrounded):
    """More than 65,536 chains: those that leave the ring kernel's 32 bits or its ring, few (a wave each) and many (rows)."""
    print(f"linear: 65,600 chains of {n} layers, {unrounded} unrounded", flush=True)
    d = inputs.uniform_aligned_chains(8, n, 65600, 256, 32768)
    at = np.random.default_rng(n).permutation(65600)[:unrounded]
    d[:, at] += inputs.uniform_aligned_chains(9, n, unrounded, 1, 9) // 4096 * (1 << 30) + 1
    d[:, at[:12]] = kinds(n, 12, 3)
    d[:, at[12:20]] = live_entries(n)  # (of 130 layers more than 64 live: the last kernel's)
    check(d)
    off = np.arange(65601, dtype=np.int64) * (n + 1)
    mask, peak, status = B.ckpt_ragged_solve_linear(torch.from_numpy(inputs.chain_major(d)).cuda().view(-1), off)
    want_peak, want_mask = oracle.batch_solve_dynamic(inputs.chain_major(d))
    assert not status.any().item()
    assert np.array_equal(peak.cpu().numpy(), want_peak)
    assert np.array_equal(mask.cpu().numpy().reshape(want_mask.shape), want_mask)


@pytest.mark.parametrize("n, large", [(16, 60000), (17, 33727), (17, 33728), (24, 47615), (24, 47616), (33, 65600), (64, 900)])
def test_large_sizes_that_the_lanes_of_a_larger_batch_leave(n, large):
    """Those of 65,600 chains that need 64 bits, on both sides of the number from which on lanes take them and not rows, a
    bad one in fifty among them."""
    print(f"linear: 65,600 chains of {n} layers, {large} with large sizes", flush=True)
    rng = np.random.default_rng(n)
    d = inputs.uniform_aligned_chains(8, n, 65600, 256, 32768)
    at = rng.permutation(65600)[:large]
    d[:, at] = rng.integers(1 << 44, (1 << 62) // (n + 2), size=(n + 1, large)) | 1
    want_peak, want_mask = oracle.batch_solve_dynamic(inputs.chain_major(d))
    want_status = np.zeros(65600, dtype=np.int32)
    for k, c in enumerate(at[::50]):
        d[k % (n + 1), c] = 0 if k % 2 else (1 << 63) - 1
        want_status[c], want_peak[c], want_mask[c] = 3 if k % 2 else 4, -1, 0
    mask, peak, status = B.ckpt_solve_linear(torch.from_numpy(d).cuda())
    assert np.array_equal(status.cpu().numpy(), want_status)
    assert np.array_equal(peak.cpu().numpy(), want_peak)
    assert np.array_equal(mask.cpu().numpy().T, want_mask)


def test_sums_at_the_ends_of_the_value_ranges():
    n, batch = 40, 1028
    rng = np.random.default_rng(5)
    for most in (1 << 30, 1 << 52):  # of sum(d) + max(d)
        d = rng.integers(1, most // (4 * n), size=(n + 1, batch)).astype(np.int64)
        for c in range(batch):
            at = (0, n // 2, n)[c % 3]
            d[(at + 1) % (n + 1), c] |= 1
            d[at, c] = (most - 2 + c % 5 - (int(d[:, c].sum()) - int(d[at, c]))) // 2
        check(d)


@pytest.mark.parametrize("batch, n", [(1024, 33), (1026, 33), (16384, 40), (16385, 40), (65536, 15), (65537, 15),
                                      (16385, 1279), (16385, 1280), (1030, 4095), (1030, 4096)])
def test_batches_on_both_sides_of_the_rules(batch, n):
    print(f"linear: {batch} chains of {n} layers", flush=True)
    d = inputs.uniform_aligned_chains(6, n, batch, 256, 32768)
    d[:, ::9] += 1
    if n < 50:
        check(d)
        return
    pick = np.r_[0:6, batch - 6:batch]  # (the oracle takes its time with the long ones)
    mask, peak, status = B.ckpt_solve_linear(torch.from_numpy(d).cuda())
    want_peak, want_mask = oracle.batch_solve_dynamic(inputs.chain_major(d[:, pick]))
    assert not status.any().item()
    assert np.array_equal(peak.cpu().numpy()[pick], want_peak)
    assert np.array_equal(mask[:, torch.from_numpy(pick).cuda()].cpu().numpy().T, want_mask)


def test_bad_chains_are_reported_alone():
    d = inputs.uniform_aligned_chains(4, 100, 1100, 256, 32768)
    want_peak, want_mask = oracle.batch_solve_dynamic(inputs.chain_major(d))
    d[100, 2] = 0
    d[0, 9] = -5
    d[:, 1098] = (1 << 62) + 3
    mask, peak, status = B.ckpt_solve_linear(torch.from_numpy(d).cuda())
    good = np.ones(1100, dtype=bool)
    good[[2, 9, 1098]] = False
    status, peak, mask = status.cpu().numpy(), peak.cpu().numpy(), mask.cpu().numpy().T
    assert (status[good] == 0).all() and (status[~good] != 0).all() and (peak[~good] == -1).all()
    assert status[2] == status[9] != status[1098]
    assert np.array_equal(peak[good], want_peak[good]) and np.array_equal(mask[good], want_mask[good])
    assert not mask[~good].any()


@pytest.mark.parametrize("batch, longest", [(5, 700), (1024, 90), (1025, 90), (4000, 300), (16385, 30), (65537, 12),
                                            (16400, 4095), (16400, 4096), (262144, 5), (262145, 5)])
def test_ragged_chains_where_they_lie(batch, longest):
    print(f"ragged linear: {batch} chains of up to {longest} layers", flush=True)
    rng = np.random.default_rng(batch)
    lengths = [int(n) for n in np.minimum(np.exp(rng.uniform(0, np.log(min(longest, 700) + 1), size=batch)), longest)]
    lengths[batch // 3] = longest
    d, _, off = inputs.ragged_batch(19, lengths)
    for c in range(0, batch, 7):  # unrounded, more than doubles hold, many live entries
        n, part = lengths[c], slice(off[c], off[c + 1])
        if c % 3 == 0:
            d[part] += 1
        elif c % 3 == 1:
            d[part] = rng.integers(1, (1 << 62) // (n + 2), size=n + 1)
        elif n > 1:
            d[part] = live_entries(n)[:, 0]
    want_peak, want_mask = oracle.ragged_solve_dynamic(d, off)
    bad = [batch // 2, batch - 1]
    for c in bad:
        d[off[c]] = 0
    for off_dev in (None, torch.from_numpy(off).cuda()):
        mask, peak, status = B.ckpt_ragged_solve_linear(torch.from_numpy(d).cuda(), off, offsets_dev=off_dev)
        mask, peak, status = mask.cpu().numpy(), peak.cpu().numpy(), status.cpu().numpy()
        for c in bad:
            assert status[c] != 0 and peak[c] == -1 and not mask[off[c]:off[c + 1]].any()
            status[c], peak[c], mask[off[c]:off[c + 1]] = 0, want_peak[c], want_mask[off[c]:off[c + 1]]
        assert (status == 0).all()
        assert np.array_equal(peak, want_peak)
        assert np.array_equal(mask, want_mask)
