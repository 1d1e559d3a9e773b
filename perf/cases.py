"""The workloads by which this library's speed is judged.

Each case is one call sequence that a user's program makes through the public entry points
(paper_2503_10302_amd.sg, paper_2503_10302_amd.ladder, the C ABI of include/sg.h), with the
sizes of the repository's benchmark, studies and tests or generic ones:

  apt        sg_run_apt_ex on a batch of instances, then the energies and spins of every replica
  apt_calls  the step-by-step calls: sweep, cluster move, swap, energies
  sqa        a DT-SQA anneal, then the energy of every slice (and the spins, where they are small)
  state      checkpoint out and in, Trotter agreement, energies and spins of a DT-SQA context
  adaptive   the adaptive inverse-temperature stage
  mlp        loss and gradient, then training epochs, of the ladder network
  learned    the learned-ladder flow: prediction, pilot runs, band check, repairs

listed() names the cases, draw() draws more of the same ranges, prepare() makes what the caller
holds beforehand, run() is one pass, work() what a pass cannot do without, exact() its results in
64 bits where they are computed numbers (the Monte Carlo results are whole numbers).
"""
import ctypes
import math

import numpy as np
import torch

from paper_2503_10302_amd import inputs, ladder, sg

# Vector operations that one spin update cannot do without: a quarter of a Philox4x32-10 block and
# a compare.
OPS_PER_FLIP = 17.4
MAX_FLIPS = 1.4e11       # of a drawn case (the largest listed anneal's)
MAX_SPIN_BYTES = 1 << 28  # spins of a whole context that are returned as bytes


def listed():
    return [
        # one small instance alone: every cycle is a chain of short dependent steps (latency)
        dict(name="apt_L8_single", kind="apt", sizes="8", periodic=7, n_inst=1, n_beta=32, reps=2, sweeps=1,
             cycles=256, record=16, cutoff=1.0, per_inst=False, pairs=2, absent=0.0, h_max=0),
        # the throughput form: a batch of instances of mixed sizes, one sweep per swap, cluster moves
        dict(name="apt_mixed_256", kind="apt", sizes="6,8,10,12,15", periodic=7, n_inst=256, n_beta=32, reps=2,
             sweeps=1, cycles=128, record=32, cutoff=1.0, per_inst=False, pairs=2, absent=0.0, h_max=0),
        # the scaling study's largest size with four labels and a cutoff per instance, and a number
        # of cycles that is no multiple of anything
        dict(name="apt_L15_labels4", kind="apt", sizes="15", periodic=7, n_inst=64, n_beta=32, reps=4, sweeps=1,
             cycles=75, record=5, cutoff=1.0, per_inst=True, pairs=2, absent=0.1, h_max=0),
        # the ablation's sweep-to-swap ratio 10 without cluster moves: long launches of plain sweeps
        dict(name="apt_L12_ratio10", kind="apt", sizes="12", periodic=7, n_inst=128, n_beta=32, reps=2, sweeps=10,
             cycles=32, record=1, cutoff=math.inf, per_inst=False, pairs=2, absent=0.0, h_max=0),
        # the smallest calls: one lattice, few temperatures, every step its own call with its results
        dict(name="apt_calls_L6", kind="apt_calls", sizes="6", periodic=7, n_inst=1, n_beta=8, reps=2, sweeps=1,
             rounds=4, cutoff=1.0, absent=0.0, h_max=0),
        # the headline anneal: 32 instances, 64 slices, 1024 replicas each
        dict(name="sqa_L15_M64_R1024", kind="sqa", sizes="15", periodic=7, n_inst=32, M=64, R=1024, beta=32.0,
             steps=20, absent=0.0, h_max=0),
        # one instance, few replicas, a schedule of several hundred steps
        dict(name="sqa_L10_M32_R64", kind="sqa", sizes="10", periodic=7, n_inst=1, M=32, R=64, beta=4.0,
             steps=600, absent=0.0, h_max=0),
        # the 15 x 15 x 12 geometry (open in x and y) with fields, a slice count between the usual ones
        dict(name="sqa_open_fields_M48", kind="sqa", sizes="15x15x12", periodic=4, n_inst=8, M=48, R=128, beta=24.0,
             steps=40, absent=0.0, h_max=2),
        # a checkpoint written and read back, and the whole state as a host program analyses it
        dict(name="sqa_state", kind="state", sizes="15", periodic=7, n_inst=4, M=32, R=64, beta=16.0,
             absent=0.0, h_max=0),
        # the adaptive stage: 100 chains per instance, a tenth of the sweeps measured
        dict(name="adaptive_L15", kind="adaptive", sizes="15", periodic=7, n_inst=64, chains=100, sweeps=1000,
             tail=100, steps=6, absent=0.0, h_max=0),
        # training of the ladder network in minibatches of 64
        dict(name="mlp_train", kind="mlp", n=2048, batch=64, epochs=4, grad_batch=256),
        # ladders for new instances: prediction, 1000-cycle pilots, repairs where a band is missed
        dict(name="learned_ladders_32", kind="learned", sizes="8,10,12,15", periodic=7, n_inst=32, pilot=1000,
             absent=0.15, h_max=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_sizes(rng, most=15):
    if rng.random() < 0.6:
        return ",".join(str(v) for v in sorted(rng.randint(4, most) for _ in range(rng.choice((1, 1, 3)))))
    return "x".join(str(rng.randint(4, most)) for _ in range(3))


def draw(rng):
    kind = rng.choice(("apt", "apt", "apt", "apt_calls", "sqa", "sqa", "sqa", "state", "adaptive", "mlp", "learned"))
    periodic = rng.choice((7, 7, 7, 4, 0))
    absent = rng.choice((0.0, 0.0, 0.1, 0.3))
    h_max = rng.choice((0, 0, 0, 1, 3))
    if kind in ("apt", "apt_calls"):
        reps = rng.choice((1, 2, 2, 4))
        icm = reps > 1 and h_max == 0 and rng.random() < 0.75
        c = dict(kind=kind, sizes=_draw_sizes(rng), periodic=periodic, n_inst=_log_int(rng, 1, 256),
                 n_beta=rng.randint(4, 40), reps=reps, sweeps=1,
                 cutoff=rng.choice((0.5, 1.0, 1.5)) if icm else math.inf, absent=absent, h_max=h_max)
        if kind == "apt_calls":
            c.update(n_inst=_log_int(rng, 1, 16), sweeps=rng.choice((1, 1, 2, 7)), rounds=rng.randint(1, 6))
            return c
        c.update(sweeps=rng.choice((1, 1, 1, 2, 10)), per_inst=icm and rng.random() < 0.3, pairs=rng.choice((1, 2, 2)),
                 cycles=_log_int(rng, 8, 300))
        c["record"] = rng.randint(1, max(1, c["cycles"] // 4))
        return c
    if kind == "sqa":
        M = rng.choice((16, 32, 64, rng.randint(2, 64), 2 * rng.randint(2, 31)))
        c = dict(kind=kind, sizes=_draw_sizes(rng), periodic=periodic, n_inst=_log_int(rng, 1, 32), M=M,
                 R=_log_int(rng, 8, 1024), beta=rng.choice((4.0, M / 2.0)), steps=_log_int(rng, 10, 600),
                 absent=absent, h_max=h_max)
        while _flips(c) > MAX_FLIPS or _spins(c) > 1 << 31:
            c["R"] = max(1, c["R"] // 2)
            c["steps"] = max(5, c["steps"] // 2)
        return c
    if kind == "state":
        c = dict(kind=kind, sizes=_draw_sizes(rng), periodic=periodic, n_inst=rng.randint(1, 4),
                 M=rng.choice((16, 32, 33, 64)), R=_log_int(rng, 4, 64), beta=8.0, absent=absent, h_max=h_max)
        while _spins(c) > 1 << 25:
            c["R"] = max(1, c["R"] // 2)
        return c
    if kind == "adaptive":
        c = dict(kind=kind, sizes=_draw_sizes(rng), periodic=periodic, n_inst=_log_int(rng, 2, 100),
                 chains=rng.choice((20, 50, 100)), sweeps=_log_int(rng, 100, 1000), tail=0, steps=rng.randint(2, 8),
                 absent=absent, h_max=h_max)
        c["tail"] = max(2, c["sweeps"] // 10)
        return c
    if kind == "mlp":
        return dict(kind=kind, n=_log_int(rng, 100, 6000), batch=rng.choice((32, 64, 64, 100)), epochs=rng.randint(1, 4),
                    grad_batch=_log_int(rng, 1, 2048))
    return dict(kind=kind, sizes=rng.choice(("8", "10", "12", "15", "8,12", "10,15")), periodic=7,
                n_inst=_log_int(rng, 1, 64), pilot=1000, absent=rng.choice((0.0, 0.1, 0.2)), h_max=0)


def _shapes(case):
    """(Lx, Ly, Lz) of every instance, the sizes in turn."""
    one = [tuple(int(v) for v in s.split("x")) for s in case["sizes"].split(",")]
    one = [s * 3 if len(s) == 1 else s for s in one]
    return [one[i % len(one)] for i in range(case["n_inst"])]


def _sites(case):
    return [s[0] * s[1] * s[2] for s in _shapes(case)]


def _instances(case, seed):
    out = []
    for i, shape in enumerate(_shapes(case)):
        J, h = inputs.ej_couplings(shape, case["periodic"], 1000 * seed + i, case["h_max"])
        if case["absent"] > 0:
            J = inputs.diluted_couplings(shape, case["periodic"], 1000 * seed + i, case["absent"])
        out.append((J, case["periodic"], h))
    return out


def _spins(case):
    """Spins that the state of a case holds."""
    k = case["kind"]
    if k in ("sqa", "state"):
        return sum(_sites(case)) * case["M"] * case["R"]
    if k in ("apt", "apt_calls"):
        return sum(_sites(case)) * case["n_beta"] * case["reps"]
    if k == "adaptive":
        return sum(_sites(case)) * case["chains"]
    return sum(_sites(case)) * 64


def _flips(case):
    """Spin updates of one pass."""
    k = case["kind"]
    per = {"apt": lambda: case["cycles"] * case["sweeps"], "apt_calls": lambda: case["rounds"] * case["sweeps"],
           "sqa": lambda: case["steps"], "adaptive": lambda: case["steps"] * case["sweeps"],
           "learned": lambda: case["pilot"], "state": lambda: 0}[k]()
    return float(_spins(case)) * per


def work(case):
    if case["kind"] == "mlp":
        # forward and backward: 2 and 4 operations per weight and sample; data and parameters once
        samples = case["n"] * case["epochs"] + case["grad_batch"]
        return {"bytes": 4.0 * (37 * (case["n"] + case["grad_batch"]) + 8 * sg.MLP_NPARAM),
                "flops": 6.0 * 6464 * samples}
    sites = sum(_sites(case))
    # the state read and written once (a bit per spin), the couplings once, and what comes back
    size = _spins(case) / 4.0 + 3.0 * sites
    if case["kind"] == "state":
        size = 4.0 * _spins(case)   # blob out and in, spins out, and the pass over them
    elif case["kind"] in ("apt", "apt_calls") or _returns_spins(case):
        size += _spins(case)
    return {"bytes": size, "flops": OPS_PER_FLIP * _flips(case)}


def _returns_spins(case):
    return case["kind"] == "sqa" and case["R"] * case["M"] * case["n_inst"] * max(_sites(case)) <= MAX_SPIN_BYTES


def _training_data(n, rng):
    """Features and targets as the adaptive stage's ladders give them: the features spread over
    the sizes and dilutions, log betas rising from about 0.2 to about 3, the cutoff near 1."""
    x = np.stack([rng.uniform(8, 15, n), rng.uniform(1.2, 1.9, n), rng.uniform(1.2, 2.4, n),
                  rng.uniform(0.46, 0.54, n)], 1)
    inc = 0.085 * np.exp(0.1 * rng.standard_normal((n, 31))) * (1.0 + 0.02 * (x[:, :1] - 12))
    y = np.empty((n, 33))
    y[:, 0] = -0.7 + 0.05 * rng.standard_normal(n)
    y[:, 1:32] = y[:, :1] + np.cumsum(inc, 1)
    y[:, 32] = 0.02 + 0.05 * rng.random(n)
    return x.astype(np.float32), y.astype(np.float32)


def _network(seed):
    """A network (W1 b1 W2 b2 W3 b3, feature mean and std) near the mean target, and its data's rng."""
    rng = np.random.default_rng([77, seed])
    parts = []
    for rows, cols, scale in ((64, 4, 0.5), (64, 64, 0.125), (33, 64, 0.0125)):
        parts += [rng.uniform(-scale, scale, (rows, cols)), rng.uniform(-scale, scale, rows)]
    parts[5] = np.r_[-0.7, np.full(31, math.log(math.expm1(0.085))), 0.05]
    stats = [np.array([11.5, 1.55, 1.8, 0.5]), np.array([2.0, 0.2, 0.35, 0.023])]
    return np.concatenate([p.reshape(-1) for p in parts + stats]).astype(np.float32), rng


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        p, rng = _network(seed)
        x, y = _training_data(case["n"], rng)
        gx, gy = _training_data(case["grad_batch"], rng)
        return dict(case=case, net=ladder.Predictor(p, seed=seed), x=x, y=y, gx=gx, gy=gy)
    inst = _instances(case, seed)
    s = dict(case=case, inst=inst, seed=seed)
    if kind in ("adaptive", "learned"):
        return s
    sites = _sites(case)
    if kind in ("sqa", "state"):
        s["ctx"] = sg.sqa(inst, case["M"], case["R"], case["beta"], seed)
        if kind == "sqa":
            s["gamma"] = inputs.linear_gamma(case["steps"])
            s["E"] = torch.zeros((case["n_inst"], case["R"], case["M"]), dtype=torch.int64, device="cuda")
            if _returns_spins(case):
                s["spins"] = torch.zeros((case["n_inst"], case["R"], case["M"], max(sites)), dtype=torch.int8,
                                         device="cuda")
        else:
            s["ctx"].sqa_anneal(inputs.linear_gamma(4))
        return s
    beta = inputs.geometric_ladder(case["n_beta"], 0.2, 3.0)
    s["ctx"] = sg.apt(inst, beta, seed, reps_per_beta=case["reps"])
    slots = case["n_beta"] * case["reps"]
    s["E"] = torch.zeros((case["n_inst"], slots), dtype=torch.int64, device="cuda")
    s["spins"] = torch.zeros((case["n_inst"], slots, max(sites)), dtype=torch.int8, device="cuda")
    s["cutoff"] = case["cutoff"]
    if case.get("per_inst"):
        s["cutoff"] = case["cutoff"] * (0.9 + 0.2 * np.random.default_rng([5, seed]).random(case["n_inst"]))
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "mlp":
        net, lib = state["net"], sg.load()
        loss, grad = ctypes.c_float(0), np.zeros(sg.MLP_NPARAM, np.float32)
        ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)   # noqa: E731
        rc = lib.sg_mlp_loss_grad(net.h, ptr(state["gx"]), ptr(state["gy"]), case["grad_batch"], ctypes.byref(loss),
                                  ptr(grad))
        if rc != sg.SG_OK:
            raise sg.SGError(rc, "sg_mlp_loss_grad")
        losses = net.train(state["x"], state["y"], epochs=case["epochs"], batch=case["batch"])
        return {"loss": np.float32(loss.value), "grad": grad, "losses": losses, "params": net.params()}
    if kind == "adaptive":
        res = sg.adaptive_ladder(state["inst"], state["seed"], n_chains=case["chains"], sweeps=case["sweeps"],
                                 tail=case["tail"], max_steps=case["steps"])
        return {"len": np.array([len(b) for b, _ in res]), "beta": np.concatenate([b for b, _ in res]),
                "sigma": np.concatenate([s for _, s in res])}
    if kind == "learned":
        lad, cut, status, acc = ladder.learned_ladders(state["inst"], state["seed"], pilot=case["pilot"])
        return {"ladders": lad, "cutoffs": cut, "status": status, "acceptance": acc}
    ctx = state["ctx"]
    if kind == "state":
        blob = ctx.get_state()
        ctx.set_state(blob)
        return {"blob": blob, "agreement": ctx.trotter_agreement(), "E": ctx.energy(), "spins": ctx.spins()}
    if kind == "sqa":
        best, best_state = ctx.sqa_anneal(state["gamma"])
        ctx.energy_dev(state["E"])
        out = {"best": best, "best_state": best_state, "E": state["E"]}
        if "spins" in state:
            ctx.spins_dev(state["spins"])
            out["spins"] = state["spins"]
        ctx.synchronize()
        return out
    out = {"E": state["E"], "spins": state["spins"]}
    if kind == "apt":
        out["trace"] = ctx.run_apt_ex(case["cycles"], case["sweeps"], state["cutoff"], case["pairs"], case["record"])
    else:
        for i in range(case["rounds"]):
            ctx.sweep(case["sweeps"])
            if math.isfinite(case["cutoff"]):
                out["icm%d" % i] = ctx.icm(state["cutoff"], want_info=True)
            out["swap%d" % i] = ctx.swap()
            out["energy%d" % i] = ctx.energy()
    ctx.energy_dev(state["E"])
    ctx.spins_dev(state["spins"])
    ctx.synchronize()
    return out


def exact(case, seed):
    if case["kind"] != "mlp":
        return None   # whole numbers, or (ladders) numbers that follow from a whole Monte Carlo run
    p, rng = _network(seed)
    _training_data(case["n"], rng)
    x, y = (a.astype(np.float64) for a in _training_data(case["grad_batch"], rng))
    p = p.astype(np.float64)
    cut = np.cumsum([0, 256, 64, 4096, 64, 2112, 33, 4, 4])
    W1, b1, W2, b2, W3, b3, mean, std = (p[a:b] for a, b in zip(cut[:-1], cut[1:]))
    W1, W2, W3 = W1.reshape(64, 4), W2.reshape(64, 64), W3.reshape(33, 64)
    xs = (x - mean) / std
    z1 = xs @ W1.T + b1
    a1 = np.maximum(z1, 0)
    z2 = a1 @ W2.T + b2
    a2 = np.maximum(z2, 0)
    o = a2 @ W3.T + b3
    out = np.concatenate([np.cumsum(np.concatenate([o[:, :1], np.logaddexp(0, o[:, 1:32])], 1), 1), o[:, 32:]], 1)
    d = out - y
    loss = np.mean(d * d)
    dy = 2 * d / d.size
    tail = np.cumsum(dy[:, 31::-1], 1)[:, ::-1]   # sum of dy_j, k <= j <= 31
    do = np.concatenate([tail[:, :1], tail[:, 1:] / (1 + np.exp(-o[:, 1:32])), dy[:, 32:]], 1)
    dz2 = (do @ W3) * (a2 > 0)
    dz1 = (dz2 @ W2) * (a1 > 0)
    grad = np.concatenate([(dz1.T @ xs).reshape(-1), dz1.sum(0), (dz2.T @ a1).reshape(-1), dz2.sum(0),
                           (do.T @ a2).reshape(-1), do.sum(0)])
    return {"loss": np.float64(loss), "grad": grad, "losses": None, "params": None}
