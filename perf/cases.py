"""The work a user of this framework has it do, as timed cases: Algorithm 1 lines 6-9 of Federated Dynamic
Averaging for K workers held as one [K, d] slab on one GPU, through FdaMonitor.

Five ways of calling it (field "call"):
  step       FdaMonitor.step: the K per-worker states, both estimates, the decision, and the synchronization
             that waits on the decision (it does not fire: the case the method is built for)
  calls      the same as three calls: local_state, estimate_variance, sync_xi
  mean       FdaMonitor.step(mean=True): the average state only
  mean_sync  the same with the average model as a by-product and a decision that always fires (Synchronous,
             Theta = 0, is this special case): the slab, w_t0, w_prev and xi are rewritten at every step
  sync       sync_xi alone, unconditional
Cases that synchronize take two slabs in turn, the workers' models of two successive rounds, because a slab
that has just been synchronized has no model change left to normalize.
"host": the program reads the decision back after every step, as a training loop that logs it does.

K, d, storage and sketch sizes are those of fda_synth.CONFIGS and of the toy training program, and sizes
between them with d off every power of two.
"""
import math

import torch

import fda_synth as S
import paper_2405_20988_amd as F

DEV = "cuda:0"
MAX_SLAB_BYTES = 5_600_000_000          # the largest configuration: 8 x 350 000 000 bf16
MAX_UPDATES = 7 * 2_800_000_000         # ... and its sketch updates, rows x workers x coordinates


def _case(name, call, K, d, dtype="f32", variants=3, l=5, m=250, host=False):
    return dict(name=name, call=call, K=K, d=d, dtype=dtype, variants=variants, l=l, m=m, host=host)


def listed():
    return [
        # the smallest configuration (5 workers of a 62K-parameter model): launches and latency
        _case("step_5x61706_f32", "step", 5, 61_706),
        # the toy training program's defaults: average state, decision read back at every step
        _case("mean_host_8x200000_f32", "mean", 8, 200_000, host=True),
        # a small model of an odd size whose workers synchronize at every step
        _case("mean_sync_11x123457_f32", "mean_sync", 11, 123_457),
        # a 2.6M-parameter model: a slab the memory-side cache holds; the calls made one by one, as bench.py does
        _case("calls_16x2600000_f32", "calls", 16, 2_600_000),
        # a 7M-parameter model, 30 workers
        _case("step_30x7000000_f32", "step", 30, 7_000_000),
        # an 18M-parameter model in bf16, odd number of workers, rows off every vector boundary
        _case("step_7x18000001_bf16", "step", 7, 18_000_001, dtype="bf16", m=500),
        # LinearFDA alone: two scalars per worker, nothing but the stream
        _case("linear_host_13x6900003_f32", "step", 13, 6_900_003, variants=1, host=True),
        # 60 workers, SketchFDA alone
        _case("step_60x20000000_f32_sketch", "step", 60, 20_000_000, variants=2, m=500),
        # the largest configuration: 350M parameters in bf16
        _case("step_8x350000000_bf16", "step", 8, 350_000_000, dtype="bf16", l=7, m=1000),
        # ... and its average state alone
        _case("mean_8x350000000_bf16", "mean", 8, 350_000_000, dtype="bf16", l=7, m=1000),
        # synchronization: every byte of the slab read and rewritten
        _case("sync_30x7000000_f32", "sync", 30, 7_000_000),
        _case("sync_8x150000001_bf16", "sync", 8, 150_000_001, dtype="bf16", l=7, m=1000),
    ]


def draw(rng):
    call = rng.choice(["step", "step", "calls", "mean", "mean_sync", "sync"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    esz = 4 if dtype == "f32" else 2
    K = int(round(math.exp(rng.uniform(math.log(2), math.log(60)))))
    # the rows and widths the sketch-size sweep covers
    l = rng.choice([3, 5, 5, 7, 9])
    m = int(round(math.exp(rng.uniform(math.log(125), math.log(2000)))))
    top = min(350_000_000, MAX_SLAB_BYTES / (K * esz), MAX_UPDATES / (K * l))
    if call in ("sync", "mean_sync"):
        top = min(top, 150_000_000, 0.25 * MAX_SLAB_BYTES / (K * esz))      # two slabs, read and written
    d = int(math.exp(rng.uniform(math.log(50_000), math.log(top))))
    variants = rng.choice([1, 2, 3, 3]) if call in ("step", "calls", "mean") else 3
    host = call in ("step", "calls", "mean") and rng.random() < 0.3
    return dict(call=call, K=K, d=d, dtype=dtype, variants=variants, l=l, m=m, host=host)


def _drift(d, heavy, gen):
    """Gaussian steps for fp32 slabs; Student-t(3) (z / sqrt(chi2_3 / 3)) for bf16 ones: the two tails of the
    named configurations."""
    z = torch.randn(d, generator=gen, device=DEV)
    if not heavy:
        return z.mul_(5e-4)
    c = torch.zeros(d, device=DEV)
    for _ in range(3):
        g = torch.randn(d, generator=gen, device=DEV)
        c.addcmul_(g, g)
    return z.div_(c.div_(3.0).sqrt_().clamp_min_(1e-20)).mul_(1e-4)


def _slab(case, centre, gen):
    w = torch.empty((case["K"], case["d"]), device=DEV,
                    dtype=torch.float32 if case["dtype"] == "f32" else torch.bfloat16)
    for k in range(case["K"]):
        w[k] = _drift(case["d"], case["dtype"] == "bf16", gen).add_(centre)
    return w


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    d, call = case["d"], case["call"]
    s = {"call": call, "host": case["host"]}
    s["w_t0"] = torch.randn(d, generator=gen, device=DEV).mul_(0.05)
    # what the workers' moves have in common; xi, the direction of the last model change, leans the same way
    shared = torch.randn(d, generator=gen, device=DEV).mul_(1e-4)
    xi = torch.randn(d, generator=gen, device=DEV).mul_(1e-4).add_(shared)
    s["xi"] = xi.div_(torch.linalg.vector_norm(xi))
    s["w_prev"] = s["w_t0"].clone()
    centre = shared.add_(s["w_t0"])
    s["slabs"] = [_slab(case, centre, gen) for _ in range(2 if call in ("sync", "mean_sync") else 1)]
    mon = F.FdaMonitor(case["K"], d, case["dtype"], case["variants"], case["l"], case["m"],
                       S.default_eps(case["m"]), S.hash_coefficients(seed, case["l"]), device=DEV)
    s["mon"] = mon
    s["by"] = "sketch" if case["variants"] & 2 else "linear"
    s["xi_arg"] = s["xi"] if case["variants"] & 1 else None
    s["theta"] = -1.0 if call == "mean_sync" else float(d)      # below, or far above, any estimate of these drifts
    s["w_bar"] = torch.empty_like(s["w_t0"]) if call == "mean_sync" else None
    # the buffers a program reads the outcome from: the state by component, the result struct
    st = mon.mean.view(1, -1) if call in ("mean", "mean_sync") else mon.state
    state = (st[:, 0], st[:, 1], st[:, 2:]) if case["variants"] & 2 else (st[:, 0], st[:, 1])
    est = (mon.est_dev[:40].view(torch.float64), mon.est_dev[40:].view(torch.int32))
    models = (*s["slabs"], s["w_t0"], s["w_prev"], s["xi"])
    s["out"] = {"sync": models, "mean_sync": state + est + models}.get(call, state + est)
    return s


def run(s):
    mon, w, w_t0, w_prev, xi = s["mon"], s["slabs"][0], s["w_t0"], s["w_prev"], s["xi_arg"]
    theta, by, host = s["theta"], s["by"], s["host"]
    est = None
    if s["call"] in ("step", "mean"):
        est = mon.step(w, w_t0, w_prev, xi, theta, decide_by=by, mean=s["call"] == "mean", want_host=host)
    elif s["call"] == "calls":
        mon.local_state(w, w_t0, xi)
        est = mon.estimate_variance(theta, want_host=host)
        if xi is not None:
            mon.sync_xi(w, w_t0, w_prev, xi, pred=by)
        else:
            mon.sync(w, w_t0, w_prev, pred=by)
    elif s["call"] == "mean_sync":
        for w in s["slabs"]:
            mon.step(w, w_t0, w_prev, xi, theta, decide_by=by, mean=True, w_bar=s["w_bar"])
    else:
        for w in s["slabs"]:
            mon.sync_xi(w, w_t0, w_prev, xi)
    if est is not None:
        return s["out"] + (est.h_linear, est.h_sketch, est.sync_linear, est.sync_sketch)
    return s["out"]


def work(case):
    K, d, lin, sk = case["K"], case["d"], case["variants"] & 1, case["variants"] & 2
    slab = K * d * (4 if case["dtype"] == "f32" else 2)
    states = 4 * (2 + (case["l"] * case["m"] if sk else 0)) * (1 if case["call"].startswith("mean") else K)
    read = slab + 4 * d + (4 * d if lin else 0)                 # rows, w_t0, xi
    per = 3 + (2 if lin else 0)                                 # drift and its square, its product with xi
    if case["call"] == "sync":
        # rows read and written, w_t0 read and written, w_prev and xi written; twice
        return {"bytes": 2 * (2 * slab + 16 * d), "flops": 2 * (K + 4) * d}
    if case["call"] == "mean_sync":
        # the state's reads, then rows, w_t0, w_prev and xi written; twice
        return {"bytes": 2 * (read + slab + 12 * d + states), "flops": 2 * (K * (per + 1) + case["l"] + 4) * d}
    if case["call"] == "mean":
        return {"bytes": read + states, "flops": (K * (per + 1) + (case["l"] if sk else 0)) * d}
    return {"bytes": read + states, "flops": K * (per + (case["l"] if sk else 0)) * d}


def tolerance(case):
    # states: fp32 drifts, sums wide enough that the drifts' own rounding is what is left
    if case["call"] in ("step", "calls", "mean"):
        return {"rel": 1e-5, "max": 1e-4}
    # models: xi is the difference of two fp32 models about 500 times its size; the mean that a bf16 row
    # stores may round the other way where its last fp32 bit differs
    return {"rel": 1e-4, "max": 1e-3} if case["dtype"] == "f32" else {"rel": 5e-4, "max": 1e-2}
