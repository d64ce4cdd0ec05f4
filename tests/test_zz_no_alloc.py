"""ckpt_solve_linear_noalloc (the entry point for callers that cannot allocate): its outputs
against ckpt_solve_linear's, bit for bit, on two calls in a row, the second on a smaller
input.  Both go through the C ABI; the outputs are tensors the test allocates beforehand."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2502_12499_amd import binding as B
from paper_2502_12499_amd import inputs
from test_gpu_linear_wave import live_entries

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_both(d_np):
    """d_np: position-major (n+1, batch).  Returns the two calls' (mask, peak, status)."""
    d = torch.from_numpy(np.ascontiguousarray(d_np)).to(DEV)
    want = B.ckpt_solve_linear(d)
    mask = torch.full_like(want[0], 7)
    peak = torch.full_like(want[1], -5)
    status = torch.full_like(want[2], -5)
    torch.cuda.synchronize()
    B.ckpt_solve_linear_noalloc(d, mask, peak, status)
    torch.cuda.synchronize()
    return want, (mask, peak, status)


def same(want, got):
    for w, g, name in zip(want, got, ("mask", "peak", "status")):
        assert torch.equal(w, g), name


def test_two_calls_in_a_row_second_smaller():
    # first call: sizes with no common power of two (every chain goes through the lists in the
    # scratch), plus chains with a size that is not positive (the second list, error statuses)
    print("noalloc call 1: 4096 chains n=64, unaligned sizes, 3 bad chains", flush=True)
    d1 = inputs.log_uniform_chains(11, 64, 4096)
    d1[5, 17] = 0
    d1[64, 400] = -3
    d1[0, 4095] = 0
    want, got = run_both(d1)
    assert int((want[2] != 0).sum()) == 3
    same(want, got)
    # second call, smaller, mixed: aligned chains (none deferred) with a few unaligned ones
    print("noalloc call 2: 1000 chains n=40, aligned sizes with 5 unaligned chains", flush=True)
    d2 = inputs.uniform_aligned_chains(12, 40, 1000, 256, 32768)
    d2[:, ::211] += 1
    want, got = run_both(d2)
    assert int((want[2] != 0).sum()) == 0
    same(want, got)


def test_limits_are_host_errors():
    lib = B.load()
    fake = ctypes.c_void_p(4096)  # never dereferenced: validation fails first
    over_batch = B.Layout(1048577, 8, 1, 1048577)
    over_n = B.Layout(4, 2048, 1, 4)
    assert lib.ckpt_solve_linear_noalloc(fake, ctypes.byref(over_batch), fake, fake, None, None) == 2
    assert lib.ckpt_solve_linear_noalloc(fake, ctypes.byref(over_n), fake, fake, None, None) == 2
    assert lib.ckpt_solve_linear_noalloc(None, ctypes.byref(B.Layout(4, 8, 1, 4)), fake, fake, None, None) == 1


def check_at_the_largest_batch(d, status):
    want = B.ckpt_solve_linear(d)
    mask, peak, code = torch.full_like(want[0], 7), torch.full_like(want[1], -5), torch.full_like(want[2], -5)
    torch.cuda.synchronize()
    B.ckpt_solve_linear_noalloc(d, mask, peak, code)
    torch.cuda.synchronize()
    assert torch.equal(code, status)
    same(want, (mask, peak, code))


def test_the_last_kernel_at_the_largest_batch():
    """With the largest batch the lists fill the library's array to its end: every chain goes through both of them (a size
    that is not positive; up to 16 layers the kernel between leaves such chains to the last one), and none may need room
    behind them."""
    n, batch = 12, 1048576
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    d = torch.randint(256, 32769, (n + 1, batch), generator=gen, device=DEV, dtype=torch.int64) * 4096
    d[n, ::2] = 1 << 50
    d[0] = 0
    check_at_the_largest_batch(d, torch.full((batch,), 3, dtype=torch.int32, device=DEV))


@pytest.mark.parametrize("bad", [11, 2000])
def test_what_rows_leave_at_the_largest_batch(bad):
    """Longer chains go to rows or a wave each, which report bad sizes themselves and leave chains with more than 64 live
    entries to the last kernel."""
    n, batch = 130, 1048576
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6)
    d = torch.randint(256, 32769, (n + 1, batch), generator=gen, device=DEV, dtype=torch.int64) * 4096
    at = torch.randperm(batch, generator=gen, device=DEV)
    d[:, at[:16]] = torch.from_numpy(live_entries(n)).to(DEV)
    status = torch.zeros(batch, dtype=torch.int32, device=DEV)
    d[n // 2, at[16:16 + bad]] = 0
    status[at[16:16 + bad]] = 3
    check_at_the_largest_batch(d, status)
    peak, mask = oracle.batch_solve_dynamic(inputs.chain_major(live_entries(n)))
    got = B.ckpt_solve_linear(d)
    assert (got[1][at[:16]] == int(peak[0])).all()
    assert (got[0][:, at[:16]] == torch.from_numpy(mask[0]).to(DEV)[:, None]).all()
