"""The calls whose speed this framework answers for.

Every case is one optimizer step of one rank's shard through the package's
public entry points, as a training loop makes it:

  scaled       zb.ShardStepCall.scaled: the prepared fused Adam step driven by
               the loss scaler (what bench.py times)
  step         zb.zero_shard_step: the fused Adam step called plainly
  split        zb.zero_shard_stats, then zb.zero_shard_apply (the seam where the
               ranks add their norms on the host)
  split_async  zb.zero_shard_stats_async, then zb.zero_shard_apply_async (the same
               seam with the sums in device memory)
  resident     zb.zero_shard_step_resident: state record and scaler on the device
  graph        one resident step captured in a HIP graph, replayed
  lamb         zb.zero_lamb_step over the shard's layer table
  lamb_split   zb.zero_shard_stats, zb.zero_lamb_moments, zb.zero_lamb_apply (layers
               that straddle shards)

`lead16` / `lead32` are the element offsets of the fp16 / fp32 arrays from an
aligned address: (0, 0) for arrays of their own; (k, 0) where the fp16 arrays
are a rank's slice of the flat gradient and parameter buffers, which starts
at rank * S for any S, while the fp32 state is the rank's own; (k, k) for a
parameter group cut out of the rank's shard.

Inputs follow the repository's workloads: parameters N(0, 0.02), warm moments
N(0, 1e-4) and |N(0, 1e-6)|, fp16 gradients N(0, 1e-3) times the loss scale
2^16.  The scale does not grow (window 0), because the gradient buffers hold
gradients of that one scale.
"""
import math

import torch

from paper_1910_02054_amd import binding as zb
from paper_1910_02054_amd import workloads

LR, BETA1, BETA2 = 1e-4, 0.9, 0.999
EPS = {"adam": 1e-8, "lamb": 1e-6}
SCALE = 2.0 ** 16
ADAM = ("scaled", "step", "split", "split_async", "resident", "graph")
LAMB = ("lamb", "lamb_split")
N_MIN, N_MAX = 1_000, 250_000_000


def _case(entry, n, lead16=0, lead32=0, wd=0.0, clip=1.0, hidden=0, mp=1, nd=1, rank=0, **kw):
    return dict(kw, entry=entry, n=n, lead16=lead16, lead32=lead32, wd=wd, clip=clip, hidden=hidden, mp=mp, nd=nd,
                rank=rank)


def listed():
    return [
        # a parameter group of biases and norms (no decay), stepped plainly: all latency
        _case("step", 9_601, lead16=1, lead32=1, name="adam_group_9k"),
        # the 4.19M-parameter workload over 4 ranks: the smallest shard of the benchmark
        _case("scaled", 1_048_576, name="adam_1m"),
        # the same shard with everything on the device, as a training iteration that never waits
        _case("resident", 1_048_576, name="adam_resident_1m"),
        # GPT-2 1.5B over 256 ranks: the usual size of a shard when many ranks share a small model
        _case("scaled", 5_859_375, wd=0.01, name="adam_5m9"),
        # the 4-rank and 256-rank shards with the norm exchanged on the device between the halves
        _case("split_async", 5_859_375, name="adam_async_5m9"),
        # 1T at MP 16 x N_d 1024, last rank: odd length, the fp16 slices at an odd flat offset
        _case("scaled", 61_034_389, lead16=3, name="adam_ragged_61m"),
        # GPT-2 1.5B over 16 ranks with the norm exchanged by the host
        _case("split", 93_750_000, name="adam_split_94m"),
        # 100B at MP 16 x N_d 25: the headline of the benchmark, the largest shard
        _case("scaled", 250_000_000, name="adam_250m"),
        # LAMB over the same shapes: many small layers, the 1.5B model's shard, the 100B model's shard
        _case("lamb", 1_048_576, wd=0.01, hidden=128, nd=4, rank=1, name="lamb_1m"),
        _case("lamb_split", 5_859_375, wd=0.01, hidden=1600, nd=256, rank=20, name="lamb_split_5m9"),
        _case("lamb", 93_750_000, wd=0.01, hidden=1600, nd=16, rank=1, name="lamb_94m"),
        _case("lamb", 250_000_000, wd=0.01, hidden=8192, mp=16, nd=25, rank=0, name="lamb_250m"),
    ]


def draw(rng):
    entry = rng.choice(ADAM + LAMB)
    n = int(math.exp(rng.uniform(math.log(N_MIN), math.log(N_MAX))))
    k = rng.choice((0, 0, 0, 0, 1, 2, 3, 5))  # half of the draws have arrays of their own
    lead16, lead32 = (k, 0) if rng.random() < 0.6 else (k, k % 4)
    c = _case(entry, n, lead16, lead32, wd=rng.choice((0.0, 0.01)), clip=rng.choice((0.0, 1.0, 1.0)))
    if entry in LAMB:
        c["hidden"], c["mp"] = rng.choice(((128, 1),) if n < 100_000 else ((128, 1), (1600, 1)) if n < 4_000_000 else
                                          ((1600, 1), (4096, 1), (8192, 16)))
        c["nd"] = rng.choice((4, 16, 25))
        c["rank"] = rng.randrange(c["nd"])
    return c


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n = case["n"]

    def out(dtype):
        lead = case["lead16"] if dtype == torch.float16 else case["lead32"]
        return torch.empty(n + 8, dtype=dtype, device="cuda")[lead:lead + n]

    def normal(std, dtype=torch.float32, positive=False):
        t = out(torch.float32).normal_(0.0, std, generator=gen)
        if positive:
            t.abs_()
        return t if dtype == torch.float32 else out(dtype).copy_(t)

    return {"g16": normal(1e-3 * SCALE, torch.float16), "master": normal(0.02), "m": normal(1e-4),
            "v": normal(1e-6, positive=True), "p16": out(torch.float16).zero_()}


def _layers(case):
    """The shard's layer table: the tensors of a GPT-2-like slice that the rank's range touches."""
    shape = workloads.ModelShape(hidden=case["hidden"], mp=case["mp"], vocab=2048 if case["hidden"] == 128 else 50257)
    lay = zb.zero_partition_layout(case["n"] * case["nd"], case["nd"], case["rank"])
    sizes = workloads.model_tensor_sizes(shape, case["n"] * case["nd"])
    return workloads.layer_offsets_in(sizes, lay.offset, lay.offset + case["n"])


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["t"] = 0
    e = case["entry"]
    arrays = [s[k] for k in ("g16", "master", "m", "v", "p16")]
    hyper = (LR, BETA1, BETA2, EPS["adam"], case["wd"])
    if e == "scaled":
        s["scaler"] = zb.Scaler(SCALE, window=0)
        s["call"] = zb.ShardStepCall([s["g16"]], *arrays[1:], *hyper, case["clip"])
    elif e == "split_async":
        s["sum"] = torch.zeros(1, dtype=torch.float64, device="cuda")
        s["skipped"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    elif e in ("resident", "graph"):
        s["record"] = zb.resident_state(arrays[0].device, *hyper, case["clip"], SCALE, window=0)
        if e == "graph":
            # one eager step on scratch arrays and a scratch record loads the kernels; the capture
            # then records the step without running it
            scratch, keep = [a.clone() for a in arrays], s["record"].clone()
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                zb.zero_shard_step_resident(*scratch, keep)
            stream.synchronize()
            zb.zero_resident_release(keep)
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"], stream=stream):
                zb.zero_shard_step_resident(*arrays, s["record"])
    elif e in LAMB:
        s["plan"] = zb.LambPlan(_layers(case))
        s["layer_sums"] = torch.zeros(2 * s["plan"].n_seg, dtype=torch.float64, device="cuda")
    return s


def run(s):
    c, e = s["case"], s["case"]["entry"]
    g, th, m, v, p = s["g16"], s["master"], s["m"], s["v"], s["p16"]
    out = {"master": th, "m": m, "v": v, "p16": p}
    s["t"] += 1
    t = s["t"]
    if e == "scaled":
        out["skipped"] = s["call"].scaled(s["scaler"])
    elif e == "step":
        out["skipped"] = zb.zero_shard_step(g, th, m, v, p, LR, BETA1, BETA2, EPS["adam"], c["wd"], t, SCALE,
                                            c["clip"])
    elif e == "split":
        total = zb.zero_shard_stats(g)
        out["skipped"] = zb.zero_shard_apply(g, th, m, v, p, total, LR, BETA1, BETA2, EPS["adam"], c["wd"], t, SCALE,
                                             c["clip"])
    elif e == "split_async":
        zb.zero_shard_stats_async(g, s["sum"])
        zb.zero_shard_apply_async(g, th, m, v, p, s["sum"], LR, BETA1, BETA2, EPS["adam"], c["wd"], t, SCALE,
                                  c["clip"], skipped=s["skipped"])
        out["sumsq"], out["skipped"] = s["sum"], s["skipped"]
    elif e == "resident":
        zb.zero_shard_step_resident(g, th, m, v, p, s["record"])
        out["record"] = s["record"]
    elif e == "graph":
        s["graph"].replay()
        out["record"] = s["record"]
    elif e == "lamb":
        out["skipped"] = zb.zero_lamb_step(s["plan"], g, th, m, v, p, LR, BETA1, BETA2, EPS["lamb"], c["wd"], t,
                                           SCALE, c["clip"])
    else:
        total = zb.zero_shard_stats(g)
        zb.zero_lamb_moments(s["plan"], g, th, m, v, total, BETA1, BETA2, EPS["lamb"], c["wd"], t, SCALE, c["clip"],
                             s["layer_sums"])
        out["skipped"] = zb.zero_lamb_apply(s["plan"], th, m, v, p, total, s["layer_sums"], LR, BETA1, BETA2,
                                            EPS["lamb"], c["wd"], t)
        out["layer_sums"] = s["layer_sums"]
    return out


def work(case):
    # gradient, parameters and moments read once; parameters, moments and fp16 copy written once
    return {"bytes": 28.0 * case["n"], "flops": (24.0 if case["entry"] in ADAM else 30.0) * case["n"]}


def tolerance(case):
    # fp32 outputs are 2.5e-8 to 6e-8 from the 64-bit values in norm.  Where another correct order of
    # operations moves fp32 parameters by one unit, about one fp16 copy in 10^4 rounds the other way,
    # by one unit of 4.9e-4 to 9.8e-4 of its value: 4e-6 to 8e-6 in norm.
    return {"rel": 1e-5, "max": 1e-3}


def exact(case, seed):
    s = _inputs(case, seed)
    n, step = case["n"], 1 << 24
    total = sum(s["g16"][a:a + step].double().square().sum() for a in range(0, n, step))
    norm = total.sqrt() / SCALE
    mult = (case["clip"] / norm if case["clip"] > 0 and norm > case["clip"] else 1.0) / SCALE
    lamb = case["entry"] in LAMB
    out = {k: torch.empty(n, dtype=torch.float64, device="cuda") for k in ("master", "m", "v")}
    u = torch.empty(n, dtype=torch.float64, device="cuda") if lamb else None
    for a in range(0, n, step):
        b = slice(a, min(n, a + step))
        g = s["g16"][b].double() * mult
        th, m, v = s["master"][b].double(), s["m"][b].double(), s["v"][b].double()
        m = BETA1 * m + (1 - BETA1) * g
        v = BETA2 * v + (1 - BETA2) * g * g
        d = (m / (1 - BETA1)) / ((v / (1 - BETA2)).sqrt() + EPS["lamb" if lamb else "adam"]) + case["wd"] * th
        out["m"][b], out["v"][b] = m, v
        out["master"][b] = th if lamb else th - LR * d
        if lamb:
            u[b] = d
    if lamb:
        off = [int(x) for x in _layers(case)]
        sums = torch.empty(2 * (len(off) - 1), dtype=torch.float64, device="cuda")
        for k, (a, b) in enumerate(zip(off, off[1:])):
            wsq, usq = out["master"][a:b].square().sum(), u[a:b].square().sum()
            sums[2 * k], sums[2 * k + 1] = wsq, usq
            out["master"][a:b] -= LR * (wsq.sqrt() / usq.sqrt()) * u[a:b]
        if case["entry"] == "lamb_split":
            out["layer_sums"] = sums
    elif case["entry"] == "split_async":
        out["sumsq"] = total.reshape(1)
    out["p16"] = out["master"]
    return out
