"""How long a call takes, for tests that compare what two calls cost."""
import torch


def shortest_us(call, tries=7, calls=8):
    """The shortest mean time of `calls` calls in a row."""
    call()
    best = float("inf")
    for _ in range(tries):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(calls):
            call()
        end.record()
        torch.cuda.synchronize()
        best = min(best, begin.elapsed_time(end) / calls * 1e3)
    return best
