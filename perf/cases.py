"""The searches that a user of this package runs, as measurable cases.

A case names a call, a shape (B instances of P workers and R iterations each, S supersteps) and whose workers they are:
``workers`` is the number of the synthetic configuration in ``workloads.CONFIGS`` whose iteration times, stragglers and
rounding the inputs follow (steady workers, stragglers, two groups rounded to 1 ms with many ties, heavy tails);
``unit`` is that of the timestamps, microseconds or nanoseconds since an epoch.  Inputs are drawn on the GPU from the
seed with the recipe of ``workloads`` (which draws on the host, one instance at a time).
"""
import math

import torch

from paper_2001_01347_amd import workloads, zipline

DEVICE = "cuda:0"
EPOCH_US = 1_700_000_000_000_000          # the timestamps of a running job count from 1970


def _case(name, call, B, P, R, workers, unit="us", S=0):
    case = {"call": call, "B": B, "P": P, "R": R, "workers": workers, "unit": unit, "S": S}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a parameter server's single decision: few workers and the paper's shortest lookahead, one call at a time
        _case("decide_16x15", "sum", 1, 16, 15, 2),
        # the same for the largest cluster of the paper's Table II: the instance is cut into windows
        _case("decide_1000x150", "sum", 1, 1000, 150, 2),
        # one decision from the workers' last iteration times alone (rows predicted inside the kernels)
        _case("decide_predicted_100x150", "predicted", 1, 100, 150, 3),
        # configuration 2: many small instances, latency and launches count
        _case("config2", "sum", 4096, 16, 64, 2),
        # configuration 3: one workgroup per instance, 2 GiB of timestamps
        _case("config3", "sum", 16384, 64, 256, 3),
        # configuration 5, the benchmark's: the largest instances, heavy tails
        _case("config5", "sum", 64, 1024, 4096, 5),
        # odd sizes and timestamps in nanoseconds, as clocks give them: spreads beyond 32 bits
        _case("nanoseconds_1021x61x241", "sum", 1021, 61, 241, 2, "ns"),
        # configuration 5's workers with the prediction folded in
        _case("predicted_config5", "predicted", 64, 1024, 4096, 5),
        # the paper's formal objective max(Z) - min(Z): small instances, and ties in windows
        _case("range_config2", "range", 4096, 16, 64, 2),
        _case("range_config4", "range", 1024, 256, 1024, 4),
        # the superstep study: 64 supersteps of 256 clusters at one of the paper's lookaheads
        _case("supersteps_64x256x16x60", "supersteps", 256, 16, 60, 2, S=64),
        # the paper's exhaustive comparator on a shape of its Table II
        _case("fullgridscan_64x100x150", "fullgridscan", 64, 100, 150, 2),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    call = rng.choice(["sum", "sum", "sum", "sum", "predicted", "predicted", "range", "range", "supersteps", "gridscan",
                       "fullgridscan"])
    workers = rng.choice([2, 3, 4, 5])
    unit = "ns" if call in ("sum", "range") and rng.random() < 0.2 else "us"
    P = _log(rng, 4, 1024)
    if call in ("gridscan", "fullgridscan"):
        # the shapes of Table II; the exhaustive scan costs P times the other
        R = _log(rng, 15, 240)
        per = P * R * (P if call == "fullgridscan" else 1)
        return _case("", call, _log(rng, 1, max(1, min(64, 90_000_000 // per))), P, R, workers)
    if call == "supersteps":
        R, S = _log(rng, 8, 240), _log(rng, 4, 64)
        return _case("", call, _log(rng, 1, max(1, min(4096, (1 << 26) // (S * P * R)))), P, R, workers, S=S)
    if rng.random() < 0.3:
        return _case("", call, 1, P, _log(rng, 8, 240), workers, unit)      # one decision at the paper's lookaheads
    most = 1 << ((20 if call == "range" else 25) if unit == "ns" else 26 if call == "range" else 28)
    R = _log(rng, 8, min(4096, most // P))
    return _case("", call, _log(rng, 1, max(1, min(16384, most // (P * R)))), P, R, workers, unit)


def _workers(case, gen):
    """Mean iteration times and start offsets of every worker, [B, P] float64 in ms."""
    cfg, B, P = workloads.CONFIGS[case["workers"]], case["B"], case["P"]

    def uniform(lo, hi):
        return lo + (hi - lo) * torch.rand(B, P, dtype=torch.float64, device=DEVICE, generator=gen)

    if cfg.bimodal:
        mean = torch.where(uniform(0.0, 1.0) >= 0.8, uniform(200.0, 300.0), uniform(90.0, 110.0))
    else:
        mean = uniform(cfg.mu_lo, cfg.mu_hi)
    slow = round(P * cfg.stragglers / cfg.P)
    if slow:
        who = uniform(0.0, 1.0).argsort(dim=1)[:, :slow]
        mean.scatter_(1, who, mean.gather(1, who) * uniform(1.5, 3.0)[:, :slow])
    offset = uniform(0.0, 1.0) * (mean if cfg.offset_hi_ms is None else cfg.offset_hi_ms)
    return mean, offset


def _ticks(ms, case, quantum):
    """float64 ms -> int64 in the case's unit, rounded to `quantum` microseconds where the configuration rounds."""
    t = (ms * (1e6 if case["unit"] == "ns" else 1e3)).round_().to(torch.int64)
    q = quantum * (1000 if case["unit"] == "ns" else 1)
    return t.add_(q // 2).div_(q, rounding_mode="floor").mul_(q) if quantum > 1 else t


def _rows(case, gen):
    """The predicted end timestamps [B, P, R], made a part of the batch at a time."""
    cfg, B, P, R = workloads.CONFIGS[case["workers"]], case["B"], case["P"], case["R"]
    mean, offset = _workers(case, gen)
    epoch = EPOCH_US * (1000 if case["unit"] == "ns" else 1)
    ts = torch.empty(B, P, R, dtype=torch.int64, device=DEVICE)
    step = max(1, (1 << 25) // (P * R))
    for b in range(0, B, step):
        n = min(step, B - b)
        if cfg.jitter == "lognormal":
            d = torch.randn(n, P, R, dtype=torch.float64, device=DEVICE, generator=gen).mul_(cfg.sigma).exp_()
        else:                                # Pareto, alpha = 3
            u = 1.0 - torch.rand(n, P, R, dtype=torch.float64, device=DEVICE, generator=gen)
            d = u.pow_(-1.0 / 3.0).mul_(cfg.sigma).add_(1.0)
        d = d.mul_(mean[b:b + n, :, None]).clamp_(min=1e-3).cumsum_(dim=2).add_(offset[b:b + n, :, None])
        ts[b:b + n] = _ticks(d, case, cfg.round_to_us).add_(epoch)
    return ts


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    call, B, P, R, S = (case[k] for k in ("call", "B", "P", "R", "S"))
    state = {"call": call, "R": R}
    if call in ("predicted", "supersteps"):
        quantum = workloads.CONFIGS[case["workers"]].round_to_us
        mean, offset = _workers(case, gen)
        state["last_end"] = _ticks(offset, case, quantum) + EPOCH_US
        if S:        # the iteration times of a worker stay similar from superstep to superstep
            mean = mean * (1.0 + 0.02 * torch.randn(S, B, P, dtype=torch.float64, device=DEVICE, generator=gen))
            quantum = 1
        state["interval"] = _ticks(mean, case, quantum).clamp_(min=1)
    else:
        state["ts"] = _rows(case, gen)
    if B == 1 and not S:
        # a server that decides barrier after barrier keeps its result buffers and its workspace
        need = {"sum": lambda: zipline.ebsp_zipline_workspace_bytes(B, P, R),
                "predicted": lambda: zipline.ebsp_predict_zipline_workspace_bytes(B, P, R),
                "range": lambda: zipline.ebsp_zipline_range_workspace_bytes(B, P, R),
                "gridscan": lambda: zipline.ebsp_gridscan_workspace_bytes(B, P, R, False),
                "fullgridscan": lambda: zipline.ebsp_gridscan_workspace_bytes(B, P, R, True)}[call]()
        third = {"range": "dmin", "gridscan": "dz", "fullgridscan": "dz"}.get(call, "wait")
        state["keep"] = {"barrier": torch.empty(B, dtype=torch.int64, device=DEVICE),
                         "iters": torch.empty(B, P, dtype=torch.int32, device=DEVICE),
                         third: torch.empty(B, dtype=torch.int64, device=DEVICE),
                         "status": torch.empty(B, dtype=torch.int32, device=DEVICE),
                         "workspace": torch.empty(max(need, 256), dtype=torch.uint8, device=DEVICE)}
    else:
        state["keep"] = {}
    return state


def run(state):
    call, keep = state["call"], state["keep"]
    if call == "sum":
        return zipline.ebsp_zipline_batch(state["ts"], **keep)
    if call == "predicted":
        return zipline.ebsp_predict_zipline_batch(state["last_end"], state["interval"], state["R"], **keep)
    if call == "range":
        return zipline.ebsp_zipline_range_batch(state["ts"], **keep)
    if call == "supersteps":
        return zipline.ebsp_simulate_supersteps(state["last_end"], state["interval"], state["R"], 2000)
    return zipline.ebsp_gridscan_batch(state["ts"], call == "fullgridscan", **keep)


def work(case):
    """Inputs once, outputs once; one subtraction, one addition and one comparison per timestamp of a search, one
    subtraction and two comparisons per (designated point, other row) of a scan."""
    call, B, P, R, S = (case[k] for k in ("call", "B", "P", "R", "S"))
    searches = max(1, S) * B
    out = searches * (20 + 4 * P)
    if call in ("predicted", "supersteps"):
        read = 8 * B * P + 8 * searches * P
    else:
        read = 8 * B * P * R
    ops = 3 * searches * P * R * (P if call == "fullgridscan" else 1)
    return {"bytes": read + out, "flops": ops}


def tolerance(case):
    """Whole numbers throughout: every correct implementation gives the same ones."""
    return "exact"
