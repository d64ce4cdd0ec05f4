"""The work that users of the checkpoint-selection solver have it do, as cases that can be timed.

`listed()` names twelve cases over the solver's real range, `draw(rng)` gives further ones of the
same ranges.  A case is prepared on the GPU from a seed (`prepare`), taken once through the public
entry points (`run`), and described by what a pass cannot do without (`work`).  All results are
exact integers, so every case's tolerance is "exact"; `exact` recomputes the smaller ones from the
plain definitions.

Sizes of a chain (field "sizes"):
  network  a bottleneck network's layer outputs (stages of three layers of widths w, w, 4w, the
           picture halved and the width doubled from stage to stage), as the ResNet-shaped chains
           of inputs.py; the seed chooses the batch size, the width and where the stages end
  aligned  4 KiB x U{256..32768}: tensor sizes as an allocator rounds them (the stress configuration)
  bytes    floor(2^(16 + 12 u)): byte counts without a common power of two (64 KiB..256 MiB)
"""
import math

import numpy as np
import torch

from paper_2502_12499_amd import binding as ckpt

DEV = "cuda"
STATUS_AND_PEAK = 12  # bytes written per chain beside its mask: one int64, one int32

# What a pass of the ranges below may cost, in the units of _cost(): no more than the listed cases.
MOST_ELEMENTS = 1048576 * 257
MOST_CUBIC = {"aligned": 4096 ** 3, "network": 4096 ** 3, "bytes": 65536 * 64 ** 3}


def listed():
    return [
        # One network, asked when its training is set up: a ResNet-152-deep chain under the model of
        # a framework that frees activations early.  The smallest call: latency and launches.
        {"name": "linear_one_network", "call": "linear", "sizes": "network", "batch": 1, "n": 152},
        # Chains with unrounded byte counts, as a search over architectures submits them by the thousand.
        {"name": "linear_bytes_batch", "call": "linear", "sizes": "bytes", "batch": 65536, "n": 64},
        # A thousand candidate partitions of a very deep network; an odd batch of long chains.
        {"name": "linear_long_batch", "call": "linear", "sizes": "aligned", "batch": 997, "n": 1001},
        # The benchmark's batch: the largest call.
        {"name": "linear_stress", "call": "linear", "sizes": "aligned", "batch": 1048576, "n": 256},
        # The peaks of given sets under both memory models, same batch.
        {"name": "eval_stress", "call": "eval", "sizes": "aligned", "batch": 1048576, "n": 256, "objective": "both"},
        # Memory per training phase of given sets (the curves that are plotted), same batch.
        {"name": "timeline_stress", "call": "timeline", "sizes": "aligned", "batch": 1048576, "n": 256,
         "objective": "static"},
        # One network under the model that keeps every checkpoint: a ResNet-152-deep one ...
        {"name": "cubic_one_network", "call": "cubic", "sizes": "network", "batch": 1, "n": 152},
        # ... a ResNet-1001-deep one ...
        {"name": "cubic_deep_network", "call": "cubic", "sizes": "network", "batch": 1, "n": 1001},
        # ... and the benchmark's long chain.
        {"name": "cubic_stress", "call": "cubic", "sizes": "aligned", "batch": 1, "n": 4096},
        # The batch of unrounded chains under that model.
        {"name": "cubic_bytes_batch", "call": "cubic", "sizes": "bytes", "batch": 65536, "n": 64},
        # Networks of the depths that Section 5 of the paper and the benchmark name, sixteen very deep
        # ones among them, in one call; the caller keeps the offsets on the device and a workspace.
        {"name": "ragged_linear_networks", "call": "ragged_linear", "sizes": "aligned", "batch": 65536,
         "lengths": "networks", "deep": 16, "offsets": "device"},
        # A graph cut into a thousand linear sub-models of any length, offsets on the host only.
        {"name": "ragged_cubic_cut_graph", "call": "ragged_cubic", "sizes": "aligned", "batch": 1000,
         "lengths": "any", "longest": 152, "offsets": "host"},
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: the calls of `listed`, batches from one chain up, n = 12 .. 1001 (4096 for the
    cubic solver), every kind of sizes, both objectives and both layouts."""
    call = rng.choice(["linear", "linear", "eval", "timeline", "cubic", "cubic", "ragged_linear", "ragged_cubic",
                       "ragged_eval"])
    sizes = rng.choice(["aligned", "aligned", "bytes"])
    if call.startswith("ragged"):
        longest = _log_uniform(rng, 24, 152 if call == "ragged_cubic" else 1001)
        case = {"call": call, "sizes": sizes, "lengths": rng.choice(["networks", "any"]),
                "offsets": rng.choice(["host", "device"])}
        if case["lengths"] == "any":
            case["longest"] = longest
        elif call == "ragged_cubic":
            case["deep"] = 0
        else:
            case["deep"] = rng.randint(0, 16)
        case["batch"] = _log_uniform(rng, 16, 1000 if call == "ragged_cubic" else 65536)
        if call == "ragged_eval":
            case["objective"] = rng.choice(["static", "dynamic", "both"])
        return case
    n = _log_uniform(rng, 12, 4096 if call == "cubic" and sizes == "aligned" else 1001)
    most = max(1, MOST_CUBIC[sizes] // n ** 3) if call == "cubic" else MOST_ELEMENTS // (n + 1)
    batch = _log_uniform(rng, 1, min(most, 65536 if call == "cubic" else 1048576))
    if batch == 1 and rng.random() < 0.5:
        sizes = "network"
    case = {"call": call, "sizes": sizes, "batch": batch, "n": n}
    if call in ("eval", "timeline"):
        case["objective"] = rng.choice(["static", "dynamic", "both"] if call == "eval" else ["static", "dynamic"])
    if batch <= 65536 and rng.random() < 0.25:
        case["chain_major"] = True
    return case


OBJECTIVE = {"static": ckpt.OBJ_STATIC, "dynamic": ckpt.OBJ_DYNAMIC, "both": ckpt.OBJ_BOTH}
WORKSPACE_OF = {"linear": ckpt.CALL_SOLVE_LINEAR, "cubic": ckpt.CALL_SOLVE_CUBIC, "eval": ckpt.CALL_EVAL_PEAK}


def _network(n, rng):
    """n + 1 layer-output sizes in bytes: input, stem, bottleneck layers in four stages, classifier."""
    batch, width, pixels = rng.randint(8, 257), 16 * rng.randint(1, 5), 8 * rng.randint(7, 29)
    ends = np.sort(rng.choice(np.arange(2, max(n - 1, 6)), size=3, replace=False))
    sizes = [batch * 4 * 3 * (2 * pixels) ** 2, batch * 4 * width * pixels ** 2]
    for k in range(2, n):
        stage = int(np.searchsorted(ends, k, side="right"))
        w, hw = width << stage, max(pixels >> stage, 1)
        sizes.append(batch * 4 * (4 * w if (k - 2) % 3 == 2 else w) * hw * hw)
    sizes.append(batch * 4 * 1000)
    return np.array(sizes[:n + 1], dtype=np.int64)


def _sizes(kind, shape, gen):
    if kind == "aligned":
        return torch.randint(256, 32769, shape, generator=gen, device=DEV, dtype=torch.int64).mul_(4096)
    out = torch.empty(shape, dtype=torch.int64, device=DEV)
    flat = out.view(-1)
    for at in range(0, flat.numel(), 1 << 26):  # (in pieces: the doubles are not kept)
        part = flat[at:at + (1 << 26)]
        u = torch.rand(part.numel(), generator=gen, device=DEV, dtype=torch.float64)
        part.copy_(torch.exp2(u.mul_(12).add_(16)).floor_())
    return out


def _lengths(case, rng):
    """The chains' lengths: the same ones for every seed, in an order that the seed chooses."""
    fixed = np.random.RandomState(case["batch"])
    if case["lengths"] == "any":  # short sub-models are the common ones
        u = fixed.uniform(math.log(2), math.log(case["longest"] + 1), size=case["batch"])
        lengths = np.minimum(np.exp(u).astype(np.int64), case["longest"])
    else:
        named = [15, 24, 152] if case["call"] == "ragged_cubic" else [15, 24, 152, 257]
        lengths = fixed.choice(np.array(named, dtype=np.int64), size=case["batch"])
        lengths[:case["deep"]] = 1001
    rng.shuffle(lengths)
    return lengths


def prepare(case, seed):
    """Sizes (and sets to evaluate) on the GPU, and the workspace that a program which calls again keeps."""
    rng = np.random.RandomState(seed % (1 << 32))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    call = case["call"]
    s = {"case": case}
    if call.startswith("ragged"):
        lengths = _lengths(case, rng)
        off = np.zeros(len(lengths) + 1, dtype=np.int64)
        np.cumsum(lengths + 1, out=off[1:])
        s["off"] = off
        s["d"] = _sizes(case["sizes"], (int(off[-1]),), gen)
        if call == "ragged_eval":
            s["mask"] = (torch.rand(int(off[-1]), generator=gen, device=DEV) < 0.25).to(torch.uint8)
            ends = torch.from_numpy(np.concatenate([off[:-1], off[1:] - 1])).to(DEV)
            s["mask"][ends] = 1
        s["off_dev"] = s["workspace"] = None
        if case["offsets"] == "device":
            which = {"ragged_linear": ckpt.CALL_SOLVE_LINEAR, "ragged_cubic": ckpt.CALL_SOLVE_CUBIC,
                     "ragged_eval": ckpt.CALL_EVAL_PEAK}[call]
            s["off_dev"] = torch.from_numpy(off).to(DEV)
            need = ckpt.load().ckpt_ragged_workspace_bytes(which, off.ctypes.data, len(lengths))
            s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        return s
    n, batch, chain_major = case["n"], case["batch"], case.get("chain_major", False)
    shape = (batch, n + 1) if chain_major else (n + 1, batch)
    if case["sizes"] == "network":
        s["d"] = torch.from_numpy(_network(n, rng).reshape(shape)).to(DEV)
    else:
        s["d"] = _sizes(case["sizes"], shape, gen)
    if call in ("eval", "timeline"):
        s["mask"] = torch.empty(shape, dtype=torch.uint8, device=DEV)
        flat = s["mask"].view(-1)
        for at in range(0, flat.numel(), 1 << 27):
            part = flat[at:at + (1 << 27)]
            part.copy_(torch.rand(part.numel(), generator=gen, device=DEV) < 0.25)
        ends = s["mask"] if not chain_major else s["mask"].t()
        ends[0] = 1
        ends[n] = 1
    else:
        need = ckpt.workspace_bytes(WORKSPACE_OF[call], ckpt.layout_of(s["d"], chain_major))
        s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    """One call; everything it returns."""
    case, d = s["case"], s["d"]
    call, major = case["call"], case.get("chain_major", False)
    if call == "linear":
        return ckpt.ckpt_solve_linear(d, chain_major=major, workspace=s["workspace"])
    if call == "cubic":
        return ckpt.ckpt_solve_cubic(d, chain_major=major, workspace=s["workspace"])
    if call == "eval":
        return ckpt.ckpt_eval_peak(d, s["mask"], OBJECTIVE[case["objective"]], chain_major=major)
    if call == "timeline":
        return ckpt.ckpt_eval_timeline(d, s["mask"], OBJECTIVE[case["objective"]], chain_major=major)
    if call == "ragged_linear":
        return ckpt.ckpt_ragged_solve_linear(d, s["off"], workspace=s["workspace"], offsets_dev=s["off_dev"])
    if call == "ragged_cubic":
        return ckpt.ckpt_ragged_solve_cubic(d, s["off"], workspace=s["workspace"], offsets_dev=s["off_dev"])
    return ckpt.ckpt_ragged_eval_peak(d, s["mask"], s["off"], OBJECTIVE[case["objective"]], workspace=s["workspace"],
                                      offsets_dev=s["off_dev"])


def work(case):
    """Every size (8 B) and mask byte read or written once, every result written once.  Operations: ten
    per position for the linear recurrence (two running maxima, two sums, the choice, the queue),
    three per cell of the cubic solver's recurrence (one sum, two comparisons), six per position
    for the evaluations."""
    call = case["call"]
    if call.startswith("ragged"):
        longest = case.get("longest", 257)
        # the mean length: of the log-uniform ones, or of the named ones
        if case["lengths"] == "any":
            n = (longest - 1) / math.log((longest + 1) / 2)
            square, cube = (longest ** 2 / 2 / math.log((longest + 1) / 2), longest ** 3 / 3 / math.log((longest + 1) / 2))
            chains = [(case["batch"], n, square, cube)]
        else:
            named = [15, 24, 152] if call == "ragged_cubic" else [15, 24, 152, 257]
            chains = [(case["batch"] / len(named), m, m ** 2, m ** 3) for m in named] + [(case["deep"], 1001, 0, 0)]
    else:
        n = case["n"]
        chains = [(case["batch"], n, n ** 2, n ** 3)]
    elements = sum(b * (n + 1) for b, n, _, _ in chains)
    values = {"both": 2}.get(case.get("objective"), 1)
    if call == "timeline":
        return {"bytes": 25 * elements + 4 * case["batch"], "flops": 6 * elements}
    if call in ("eval", "ragged_eval"):
        return {"bytes": 9 * elements + (8 * values + 4) * case["batch"], "flops": 6 * elements}
    if call in ("linear", "ragged_linear"):
        return {"bytes": 9 * elements + STATUS_AND_PEAK * case["batch"], "flops": 10 * elements}
    cells = sum(b * ((cube - square) / 2 + n) for b, n, square, cube in chains)
    return {"bytes": 9 * elements + (8 + STATUS_AND_PEAK) * case["batch"], "flops": 3 * cells}


def tolerance(case):
    return "exact"  # whole bytes and sets: nothing is rounded, and ties have one canonical answer


def exact(case, seed):
    """The same results from the definitions, in plain torch on 64-bit integers: the running sums of
    the evaluations, the dynamic recurrence with every successor tried, the static recurrence with
    every budget and predecessor tried.  None where that takes too long, and for ragged calls
    (whose chains get what they get on their own)."""
    call = case["call"]
    if call.startswith("ragged") or call == "timeline":
        return None
    n, batch = case["n"], case["batch"]
    tried = {"eval": n, "linear": n * n * 8, "cubic": n ** 4}[call]
    if tried * batch > 1e10 or n > 300:
        return None
    s = prepare(case, seed)
    major = case.get("chain_major", False)
    d = s["d"].t().contiguous() if major else s["d"]
    status = torch.zeros(batch, dtype=torch.int32, device=DEV)
    if call == "eval":
        m = (s["mask"].t() if major else s["mask"]).bool()
        zero = torch.zeros(batch, dtype=torch.int64, device=DEV)
        kept, seg, seg_max, worst, peak = d[0].clone(), zero.clone(), d[0].clone(), zero.clone(), zero.clone()
        for k in range(1, n + 1):
            on, x = m[k], d[k]
            kept = torch.where(on, kept + x, kept)
            worst = torch.where(on, torch.maximum(worst, seg), worst)
            peak = torch.where(on, torch.maximum(peak, kept + seg + seg_max), peak)
            seg_max = torch.where(on, x, torch.maximum(seg_max, x))
            seg = torch.where(on, zero, seg + x)
        rows = {"static": kept + worst, "dynamic": peak}
        got = torch.stack([rows["static"], rows["dynamic"]]) if case["objective"] == "both" else rows[case["objective"]]
        return got, status
    mask = torch.zeros_like(d, dtype=torch.uint8)
    at = torch.arange(batch, device=DEV)
    if call == "linear":
        M, nxt = [None] * n + [d[n].clone()], torch.zeros_like(d)
        for i in range(n - 1, -1, -1):
            best = torch.full((batch,), 1 << 62, dtype=torch.int64, device=DEV)
            inside, top = torch.zeros(batch, dtype=torch.int64, device=DEV), d[i].clone()
            for j in range(i + 1, n + 1):
                inside = inside + d[j]
                v = torch.maximum(M[j], inside + top)
                nxt[i] = torch.where(v < best, j, nxt[i])
                best = torch.minimum(best, v)
                top = torch.maximum(top, d[j])
            M[i] = d[i] + best
        here = torch.zeros(batch, dtype=torch.int64, device=DEV)
        for k in range(n + 1):
            mask[k] = (here == k).to(torch.uint8)
            here = torch.where(here == k, nxt[k], here)
        mask[n] = 1
        return (mask.t().contiguous() if major else mask), M[0], status
    P = torch.cumsum(d, 0)
    pairs = [(a, b) for a in range(1, n) for b in range(a, n)]
    a, b = (torch.tensor([p[k] for p in pairs] or [0], device=DEV) for k in (0, 1))
    zero = torch.zeros((1, batch), dtype=torch.int64, device=DEV)
    s_all = torch.cat([zero, P[b] - P[a - 1]]) if pairs else zero

    def costs(budgets, want_pred=False):
        F, pred = [d[0].expand_as(budgets)], [None]
        for j in range(1, n + 1):
            best = torch.full_like(budgets, 1 << 62)
            of = torch.zeros_like(budgets)
            for h in range(j):
                v = torch.where(P[j - 1] - P[h] <= budgets, F[h], 1 << 62)
                if want_pred:
                    of = torch.where(v < best, h, of)
                best = torch.minimum(best, v)
            F.append(d[j] + best)
            pred.append(of)
        return F[n], pred

    total = torch.cat([costs(part)[0] + part for part in s_all.split(max(1, (1 << 25) // batch))])
    peak = total.min(0).values
    budget = torch.where(total == peak, s_all, 1 << 62).min(0).values
    _, pred = costs(budget[None], True)
    here = torch.full((batch,), n, dtype=torch.int64, device=DEV)
    for k in range(n, -1, -1):
        on = here == k
        mask[k] = on.to(torch.uint8)
        if k:
            here = torch.where(on, pred[k][0], here)
    return (mask.t().contiguous() if major else mask), peak, budget, status
