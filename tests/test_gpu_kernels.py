"""GPU parity of single kernels at the edges of their tiles, bit for bit against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2503_10302_amd import sg
from paper_2503_10302_amd.inputs import diluted_couplings, ej_couplings, geometric_ladder

pytestmark = pytest.mark.gpu
SEED = 0x0DD_5EED


def _apt_cycles_match(insts, reps, cycles, cutoff, sweeps=1, n_beta=4):
    """run_apt and one further cluster move with its records, spins and energies compared."""
    beta = geometric_ladder(n_beta, 0.2, 3.0)
    ctx = sg.apt(insts, beta, SEED, reps_per_beta=reps)
    trace = ctx.run_apt(cycles, sweeps, cutoff, record_every=1)
    icm = np.isfinite(cutoff)
    info = ctx.icm(cutoff, want_info=True) if icm else None
    spins, E = ctx.spins(), ctx.energy()
    for i, inst in enumerate(insts):
        lat = oracle.Lattice(*inst)
        sp = oracle.apt_init(lat, i, n_beta * reps, SEED)
        ctr, oE = np.zeros(3, np.uint32), np.zeros(n_beta * reps, np.int64)
        best = np.array([np.iinfo(np.int64).max], np.int64)
        rc, otr, _ = oracle.apt_run(lat, i, beta, reps, SEED, cycles, sweeps, cutoff, 1, ctr, sp, oE, best)
        assert rc == 0 and np.array_equal(trace[i], otr), f"trace, instance {i}"
        if icm:
            rc, oinfo = oracle.apt_icm(lat, i, beta, reps, cutoff, SEED, cycles + 1, sp)
            assert rc == 0 and np.array_equal(info[i], oinfo), f"records, instance {i}"
        assert np.array_equal(spins[i, :, :lat.n], sp), f"spins, instance {i}"
        assert E[i].tolist() == [oracle.energy(lat, s) for s in sp], f"energies, instance {i}"


@pytest.mark.parametrize("reps", [2, 4])
def test_one_wave_cluster_search_shapes(reps):
    """Every number of planes per lane (lz 1..16), rows at both halves' ends, axes of one and two
    sites, open axes and missing bonds, in one context of lattices of at most 16 sites an axis."""
    shapes = [(16, 16, 16), (2, 16, 5), (16, 1, 13), (5, 2, 4), (3, 3, 9), (1, 7, 16), (15, 15, 12),
              (8, 8, 1), (9, 16, 8), (4, 5, 2), (1, 1, 3)]
    insts = [(ej_couplings(s, p, 40 + i)[0], p, None)
             for i, s in enumerate(shapes) for p in ((7,) if i % 2 else (7, 5))]
    insts += [(diluted_couplings(s, 7, 80 + i, 0.25), 7, None) for i, s in enumerate(shapes[:4])]
    _apt_cycles_match(insts, reps, 3, 0.3)


@pytest.mark.parametrize("shape,n_inst,h_max", [((10, 10, 10), 1, 0), ((13, 13, 13), 1, 0), ((15, 15, 15), 70, 0),
                                                ((16, 16, 9), 2, 3)])
def test_larger_work_groups(shape, n_inst, h_max):
    """The replica kernel's 512- and 1024-thread forms (few work-groups, phases of several passes):
    a graph of cycles and single ones, with cluster moves or with fields."""
    insts = [ej_couplings(shape, 7, 60 + i, h_max=h_max) for i in range(n_inst)]
    insts = [(J, 7, h) for J, h in insts]
    _apt_cycles_match(insts[:3] if n_inst < 4 else insts, 2, 34 if n_inst < 4 else 2,
                      float("inf") if h_max else 0.5)


@pytest.mark.parametrize("batch", [1, 63, 64, 65, 130, 8192, 8193])
def test_mlp_gradient_batch_edges(batch):
    """Loss and gradient at the edges of the summation groups and of the record chunks against the
    FP64 oracle.  FP32 sums of n terms are off by at most about n 2^-24 of their absolute sum (in
    practice by its square root); 2e-5 of the largest entry leaves a factor of some ten."""
    import ctypes as C
    from paper_2503_10302_amd import ladder
    rng = np.random.default_rng(batch)
    net = ladder.Predictor(seed=3)
    p = net.params()
    x = rng.standard_normal((batch, 4)).astype(np.float32)
    y = rng.standard_normal((batch, 33)).astype(np.float32)
    loss, grad = C.c_float(0), np.zeros(sg.MLP_NPARAM, np.float32)
    rc = net.lib.sg_mlp_loss_grad(net.h, x.ctypes.data_as(C.c_void_p), y.ctypes.data_as(C.c_void_p), batch,
                                  C.byref(loss), grad.ctypes.data_as(C.c_void_p))
    assert rc == 0
    oloss, ograd, _ = oracle.mlp_loss_grad(p[:sg.MLP_NPARAM].astype(np.float64), x, y)
    assert abs(loss.value - oloss) <= 1e-5 * abs(oloss)
    assert np.abs(grad - ograd).max() <= 2e-5 * np.abs(ograd).max()


@pytest.mark.parametrize("shape,n_inst,n_chains", [((3, 4, 2), 520, 8), ((3, 4, 2), 520, 11), ((4, 3, 3), 520, 16),
                                                   ((2, 3, 4), 520, 20), ((3, 4, 2), 520, 24), ((3, 3, 2), 520, 25),
                                                   ((3, 4, 2), 520, 32), ((3, 2, 2), 300, 100),
                                                   ((12, 12, 12), 12, 100)])
def test_adaptive_word_splits(shape, n_inst, n_chains):
    """Every number of groups per chain word of the adaptive kernel (2 to 8, words with one group
    less beside them, a last group that is not full) and its 1024-thread form."""
    insts = [(ej_couplings(shape, 7, 300 + i)[0], 7, None) for i in range(n_inst)]
    kw = dict(beta0=0.4, alpha=1.25, tol=0.01, n_chains=n_chains, sweeps=5, tail=3, max_steps=2)
    got = sg.adaptive_ladder(insts, 21, **kw)
    for i in range(0, n_inst, max(1, n_inst // 40)):
        beta, sigma = oracle.adaptive_ladder(oracle.Lattice(*insts[i]), i, 21, **kw)[:2]
        assert np.array_equal(got[i][0], beta) and np.array_equal(got[i][1], sigma), f"instance {i}"


@pytest.mark.parametrize("h_max", [0, 12])
@pytest.mark.parametrize("M", [4, 9, 12, 17, 20, 25, 28, 36, 41, 44, 49, 52, 57, 60, 61])
def test_sqa_group_counts(M, h_max):
    """Every number of slice groups per word, even and odd M (with the last slice alone in its
    group at M = 9, 17, ...), in the scaled (no fields) and the unscaled table form."""
    inst = []
    for i, (shape, periodic) in enumerate([((4, 3, 2), 7), ((3, 3, 3), 5)]):
        J, h = ej_couplings(shape, periodic, 500 + i, h_max=h_max)
        inst.append((J, periodic, h))
    gam = np.linspace(3.0, 0.1, 5)
    ctx = sg.sqa(inst, M, 2, 3.0, SEED)
    bE, bs = ctx.sqa_anneal(gam)
    spins, E = ctx.spins(), ctx.energy()
    for i, x in enumerate(inst):
        lat = oracle.Lattice(*x)
        sp = oracle.sqa_init(lat, i, M, 2, SEED)
        oE, ostate, _ = oracle.sqa_anneal(lat, i, M, 2, 3.0, gam, SEED, 0, sp)
        assert np.array_equal(spins[i, :, :, :lat.n], sp) and bE[i] == oE, f"instance {i}"
        assert np.array_equal(bs[i, :lat.n], ostate)
        assert E[i].min() == oE


@pytest.mark.parametrize("steps", [128, 129, 289])
def test_sqa_schedule_in_launches(steps):
    """A schedule whose launches (32, 256 and remaining steps) take their own threshold tables."""
    J, h = ej_couplings((3, 2, 2), 7, 520, h_max=1)
    gam = np.linspace(3.0, 0.1, steps)
    ctx = sg.sqa([(J, 7, h)], 6, 2, 3.0, SEED)
    bE, _ = ctx.sqa_anneal(gam)
    lat = oracle.Lattice(J, 7, h)
    sp = oracle.sqa_init(lat, 0, 6, 2, SEED)
    oE, _, _ = oracle.sqa_anneal(lat, 0, 6, 2, 3.0, gam, SEED, 0, sp)
    assert np.array_equal(ctx.spins()[0], sp) and bE[0] == oE


@pytest.mark.parametrize("mode", ["apt", "sqa"])
@pytest.mark.parametrize("shapes", [[(1, 1, 1)], [(3, 1, 1), (5, 7, 3)], [(15, 15, 15), (4, 4, 4), (11, 9, 13)]])
def test_spins_in_and_out(mode, shapes):
    """Spins written and read back through the device packing at odd row lengths: small states (checked
    on the host) and large ones (checked on the device, several staging buffers), parts of an
    instance, and a state with one bad byte refused unchanged."""
    insts = [(ej_couplings(s, 7, 700 + i)[0], 7, None) for i, s in enumerate(shapes)]
    n_max, big = max(int(np.prod(s)) for s in shapes), len(shapes) == 3
    if mode == "apt":
        ctx = sg.apt(insts, geometric_ladder(5, 0.2, 3.0), SEED, reps_per_beta=2)
        lead = (10,)
    else:
        R = 310 if big else 3      # 3 x 310 x 33 x 3375 spins: 104 MB
        ctx = sg.sqa(insts, 33, R, 2.0, SEED)
        lead = (R, 33)
    rng = np.random.default_rng(1)
    s = np.zeros((len(insts), *lead, n_max), np.int8)
    for i, shape in enumerate(shapes):
        n = int(np.prod(shape))
        s[i, ..., :n] = 2 * rng.integers(0, 2, (*lead, n), dtype=np.int8) - 1
    ctx.set_spins(s)
    assert np.array_equal(ctx.spins(), s)
    last = len(insts) - 1
    n = int(np.prod(shapes[last]))
    assert np.array_equal(ctx.spins_range(last, 1, 2), s[last, 1:3, ..., :n])
    if mode == "apt":
        lat = oracle.Lattice(*insts[0])
        assert ctx.energy()[0].tolist() == [oracle.energy(lat, v[:lat.n]) for v in s[0]]
    for value in (0, 2, -2, 127, -128):
        bad = s.copy()
        bad[last, ..., n - 1].flat[-1] = value
        with pytest.raises(sg.SGError):
            ctx.set_spins(bad)
    assert np.array_equal(ctx.spins(), s)
    bad = s.copy()
    if n < n_max:
        bad[last, ..., n:] = 7     # bytes past an instance's sites are not looked at
        ctx.set_spins(bad)
        assert np.array_equal(ctx.spins(), s)


@pytest.mark.parametrize("shape,n_inst,n_beta,reps,S,cutoff", [
    ((3, 4, 2), 520, 8, 1, 2, float("inf")), ((4, 3, 3), 520, 11, 1, 3, float("inf")),
    ((2, 3, 4), 520, 4, 4, 2, float("inf")), ((3, 4, 2), 520, 10, 2, 5, 1.0),
    ((3, 3, 2), 520, 12, 2, 6, 0.5), ((4, 2, 2), 520, 7, 4, 5, 1.0), ((3, 4, 2), 520, 15, 2, 2, float("inf")),
    ((2, 2, 3), 300, 25, 4, 2, float("inf")), ((12, 12, 12), 12, 25, 4, 2, float("inf")),
    ((5, 7, 3), 520, 16, 2, 5, 1.0)])
def test_sweeps_in_words(shape, n_inst, n_beta, reps, S, cutoff):
    """Several sweeps per cycle in words of 2 to 8 quads of slots (the last quad not full, words with
    one quad less beside them, 512 and 1024 threads), cluster moves in launches of their own: a graph
    of cycles, single ones and a sweep call."""
    insts = [(ej_couplings(shape, 7, 800 + i)[0], 7, None) for i in range(n_inst)]
    beta = geometric_ladder(n_beta, 0.2, 3.0)
    cycles = 33 if np.prod(shape) < 200 else 2
    ctx = sg.apt(insts, beta, SEED, reps_per_beta=reps)
    trace = ctx.run_apt(cycles, S, cutoff, record_every=1)
    ctx.sweep(3)
    spins, E, counts = ctx.spins(), ctx.energy(), ctx.swap_counts()
    for i in range(0, n_inst, max(1, n_inst // 24)):
        lat = oracle.Lattice(*insts[i])
        sp = oracle.apt_init(lat, i, n_beta * reps, SEED)
        ctr, oE = np.zeros(3, np.uint32), np.zeros(n_beta * reps, np.int64)
        best = np.array([np.iinfo(np.int64).max], np.int64)
        rc, otr, oacc = oracle.apt_run(lat, i, beta, reps, SEED, cycles, S, cutoff, 1, ctr, sp, oE, best)
        assert rc == 0 and np.array_equal(trace[i], otr) and np.array_equal(counts[i], oacc), f"instance {i}"
        for k in range(3):
            oracle.apt_sweep(lat, i, np.repeat(beta, reps), SEED, cycles * S + k, sp)
        assert np.array_equal(spins[i], sp), f"spins, instance {i}"
        assert E[i].tolist() == [oracle.energy(lat, v) for v in sp], f"energies, instance {i}"


@pytest.mark.parametrize("code", [0, 14])
def test_calls_and_short_runs_interleaved(code):
    """Single calls (whose steps the device counters learn of later) between runs of every kind of
    length, in one and two launch groups, with a checkpoint taken in between."""
    insts = [(ej_couplings(s, 7, 900 + i)[0], 7, None) for i, s in enumerate([(5, 4, 3), (4, 4, 4), (3, 3, 3)])]
    beta, reps = geometric_ladder(6, 0.3, 2.5), 2
    ctx = sg.apt(insts, beta, SEED, reps_per_beta=reps)
    ctx.set_launch_config(code)
    lats = [oracle.Lattice(*x) for x in insts]
    sps = [oracle.apt_init(lat, i, 12, SEED) for i, lat in enumerate(lats)]
    ctr = np.zeros((3, 3), np.uint32)
    Es = [np.array([oracle.energy(lat, v) for v in sp], np.int64) for lat, sp in zip(lats, sps)]
    best = [np.array([np.iinfo(np.int64).max], np.int64) for _ in lats]

    def check(what):
        g, E, b = ctx.spins(), ctx.energy(), ctx.best()
        assert ctx.counters().tolist() == ctr[0].tolist(), what
        for i, lat in enumerate(lats):
            assert np.array_equal(g[i, :, :lat.n], sps[i]), f"{what}, spins {i}"
            assert E[i].tolist() == [oracle.energy(lat, v) for v in sps[i]], f"{what}, energies {i}"
            assert ctr[0, 2] == 0 or b[i] == best[i][0], f"{what}, minimum {i}"

    for step, n in enumerate((1, 2, 3, 31, 33, 5, 64, 34)):
        ctx.sweep(2)
        ctx.icm(0.8)
        acc = ctx.swap()
        trace = ctx.run_apt(n, 1, 0.8, record_every=1)
        for i, lat in enumerate(lats):
            for k in range(2):
                oracle.apt_sweep(lat, i, np.repeat(beta, reps), SEED, int(ctr[i, 0]) + k, sps[i])
            oracle.apt_icm(lat, i, beta, reps, 0.8, SEED, int(ctr[i, 1]) + 1, sps[i])
            Es[i][:] = [oracle.energy(lat, v) for v in sps[i]]
            oacc = oracle.apt_swap(i, beta, reps, SEED, int(ctr[i, 2]) + 1, sps[i], Es[i])
            assert np.array_equal(acc[i], oacc)
            best[i][0] = min(best[i][0], Es[i].min())
            ctr[i] += np.array([2, 1, 1], np.uint32)
            rc, otr, _ = oracle.apt_run(lat, i, beta, reps, SEED, n, 1, 0.8, 1, ctr[i], sps[i], Es[i], best[i])
            assert rc == 0 and np.array_equal(trace[i], otr), f"trace of {n} cycles, instance {i}"
        check(f"after {n} cycles")
        if step == 3:
            ctx.sweep(1)
            blob = ctx.get_state()
            ctx.sweep(3)
            ctx.set_state(blob)
            for i, lat in enumerate(lats):
                oracle.apt_sweep(lat, i, np.repeat(beta, reps), SEED, int(ctr[i, 0]), sps[i])
                ctr[i, 0] += 1
            check("after the checkpoint")


def _hip():
    """The HIP runtime that libsg itself uses."""
    import ctypes
    sg.load()
    return ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))


@pytest.mark.parametrize("shapes,n_beta,reps,sweeps", [([(5, 4, 3), (4, 4, 4)], 6, 2, 1),
                                                       ([(12, 12, 12)] * 12, 25, 4, 12)])
def test_captured_calls_replay_with_new_random_numbers(monkeypatch, shapes, n_beta, reps, sweeps):
    """Sweeps, cluster moves and an exchange, recorded by the caller into a graph on the stream it
    gave the context (the sweeps in tiles and in words), then replayed between calls of its own:
    every replay takes the next step numbers."""
    import ctypes as C
    hip = _hip()
    stream = C.c_void_p()
    assert hip.hipStreamCreateWithFlags(C.byref(stream), 1) == 0
    config = sg._Config
    monkeypatch.setattr(sg, "_Config", lambda *a: config(*a[:-1], stream))
    insts = [(ej_couplings(s, 7, 950 + i)[0], 7, None) for i, s in enumerate(shapes)]
    beta = geometric_ladder(n_beta, 0.3, 2.5)
    cut = float(beta[-2])

    def steps(c):
        c.sweep(sweeps)
        c.icm(cut)
        c.swap(want_flags=False)

    twin = sg.apt(insts, beta, SEED + 1, reps_per_beta=reps)
    steps(twin)   # the kernels are loaded
    twin.close()
    ctx = sg.apt(insts, beta, SEED, reps_per_beta=reps)
    ctx.set_launch_config(1)
    ctx.icm(cut)  # the flags of this cutoff are on the device
    ctx.swap()
    graph, replay = C.c_void_p(), C.c_void_p()
    assert hip.hipStreamBeginCapture(stream, 1) == 0
    steps(ctx)
    assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
    assert hip.hipGraphInstantiate(C.byref(replay), graph, None, None, C.c_size_t(0)) == 0

    pick = sorted({0, len(insts) - 1})
    lats = {i: oracle.Lattice(*insts[i]) for i in pick}
    sps = {i: oracle.apt_init(lats[i], i, n_beta * reps, SEED) for i in pick}
    ctr = [0, 0, 0]

    def oracle_icm():
        for i in pick:
            oracle.apt_icm(lats[i], i, beta, reps, cut, SEED, ctr[1] + 1, sps[i])
        ctr[1] += 1

    def oracle_swap():
        for i in pick:
            E = np.array([oracle.energy(lats[i], v) for v in sps[i]], np.int64)
            oracle.apt_swap(i, beta, reps, SEED, ctr[2] + 1, sps[i], E)
        ctr[2] += 1

    def oracle_sweeps(n):
        for i in pick:
            for k in range(n):
                oracle.apt_sweep(lats[i], i, np.repeat(beta, reps), SEED, ctr[0] + k, sps[i])
        ctr[0] += n

    oracle_icm()
    oracle_swap()
    for k in range(3):
        assert hip.hipGraphLaunch(replay, stream) == 0
        oracle_sweeps(sweeps)
        oracle_icm()
        oracle_swap()
        assert ctx.counters().tolist() == ctr, f"replay {k}"
        spins, E = ctx.spins(), ctx.energy()
        for i in pick:
            assert np.array_equal(spins[i, :, :lats[i].n], sps[i]), f"replay {k}, spins {i}"
            assert E[i].tolist() == [oracle.energy(lats[i], v) for v in sps[i]], f"replay {k}, energies {i}"
        # calls, a run (graph and single cycles) and a checkpoint of the caller's own between the replays
        ctx.sweep(1)
        oracle_sweeps(1)
        ctx.run_apt(33, 1, cut)
        for _ in range(33):
            oracle_sweeps(1)
            oracle_icm()
            oracle_swap()
        blob = ctx.get_state()
        ctx.sweep(3)
        ctx.swap()
        ctx.set_state(blob)
    assert hip.hipGraphExecDestroy(replay) == 0 and hip.hipGraphDestroy(graph) == 0
    ctx.close()
    assert hip.hipStreamDestroy(stream) == 0


def test_runs_in_words_leave_the_launch_configuration_unset():
    """A first run whose sweeps are in words, without and with cluster moves, leaves the choice to the
    first run in tiles, which tunes its own shape; a code that is set stays."""
    insts = [(ej_couplings((8, 8, 8), 7, 970 + i)[0], 7, None) for i in range(64)]
    beta = geometric_ladder(64, 0.2, 3.0)
    ctx = sg.apt(insts, beta, SEED, reps_per_beta=4)
    for cutoff in (float("inf"), 1.0):
        ctx.run_apt(34, 12, cutoff)
        assert ctx.launch_config() == 0
    ctx.run_apt(2, 1, 1.0)
    assert 1 <= ctx.launch_config() <= 15
    ctx.set_launch_config(13)
    ctx.run_apt(2, 12, 1.0)
    assert ctx.launch_config() == 13
    lat, sp = oracle.Lattice(*insts[63]), oracle.apt_init(oracle.Lattice(*insts[63]), 63, 256, SEED)
    ctr, E = np.zeros(3, np.uint32), np.zeros(256, np.int64)
    best = np.array([np.iinfo(np.int64).max], np.int64)
    for cycles, sweeps, cutoff in ((34, 12, float("inf")), (34, 12, 1.0), (2, 1, 1.0), (2, 12, 1.0)):
        rc, _, _ = oracle.apt_run(lat, 63, beta, 4, SEED, cycles, sweeps, cutoff, 1, ctr, sp, E, best)
        assert rc == 0
    assert np.array_equal(ctx.spins()[63], sp) and ctx.energy()[63].tolist() == E.tolist()


@pytest.mark.parametrize("shapes,n_inst,n_beta,reps,sweeps,cutoff,words", [
    ([(8, 8, 8)], 64, 32, 2, 2, float("inf"), False), ([(5, 5, 5)], 100, 32, 2, 10, float("inf"), False),
    ([(15, 15, 15)], 32, 32, 2, 2, float("inf"), False), ([(15, 15, 15), (6, 6, 6)], 40, 20, 2, 10, float("inf"), False),
    ([(12, 12, 12)], 64, 32, 2, 5, 1.0, False), ([(5, 5, 5)], 100, 32, 2, 10, 1.0, False),
    ([(12, 12, 12)], 128, 32, 2, 2, float("inf"), True), ([(15, 15, 15)], 32, 32, 2, 10, float("inf"), True),
    ([(12, 12, 12)], 128, 32, 2, 10, 1.0, True), ([(20, 20, 20)], 8, 32, 2, 2, float("inf"), True)])
def test_sweeps_run_in_words_where_they_pay(shapes, n_inst, n_beta, reps, sweeps, cutoff, words):
    """The choice between words and tiles on batches on both sides of the line, each with its measured
    winner.  (Only a run in tiles settles the launch configuration.)"""
    insts = [(ej_couplings(shapes[i % len(shapes)], 7, 1000 + i)[0], 7, None) for i in range(n_inst)]
    ctx = sg.apt(insts, geometric_ladder(n_beta, 0.2, 3.0), SEED, reps_per_beta=reps)
    ctx.run_apt(2, sweeps, cutoff)
    assert (ctx.launch_config() == 0) == words


_MIXED_WORDS = [(5, 4, 3), (4, 4, 4), (3, 5, 2), (6, 3, 4), (1, 1, 3), (7, 6, 5), (2, 2, 2), (9, 4, 2)]
_MIXED_AXES = [7, 7, 5, 7, 0, 3, 7, 6]   # periodic axes of each


@pytest.mark.parametrize("shapes,n_inst,n_beta,reps,S,cutoff", [
    ([(8, 8, 8)], 64, 32, 2, 20, float("inf")), ([(12, 12, 12)], 12, 25, 4, 6, float("inf")),
    ([(3, 4, 2)], 1500, 11, 1, 3, float("inf")), ([(4, 3, 3)], 1500, 16, 1, 4, float("inf")),
    ([(2, 3, 4)], 1500, 20, 1, 2, float("inf")), ([(3, 4, 2)], 1500, 12, 2, 5, 1.0),
    ([(3, 3, 2)], 1500, 14, 2, 5, 0.5), ([(4, 2, 2)], 1500, 8, 4, 5, 1.0), ([(3, 4, 2)], 1500, 9, 4, 2, float("inf")),
    ([(2, 2, 3)], 1500, 13, 4, 5, 1.0), (_MIXED_WORDS, 800, 15, 4, 5, 1.0), ([(18, 18, 18)], 130, 8, 4, 2, float("inf")),
    ([(22, 21, 23)], 4, 8, 2, 2, float("inf"))])
def test_words_of_every_size(shapes, n_inst, n_beta, reps, S, cutoff):
    """Batches whose sweeps run in words: 2 to 8 groups of four slots in the fuller words, words with one
    group less beside them, 512 and 1024 threads; mixed sizes with open axes and missing bonds; and the
    wide bond counters of lattices with more than ten sites per thread."""
    insts = []
    for i in range(n_inst):
        k = i % len(shapes)
        per = _MIXED_AXES[k] if len(shapes) > 1 else 7
        diluted = len(shapes) > 1 and (i // len(shapes)) % 2
        J = diluted_couplings(shapes[k], per, 1100 + i, 0.25) if diluted else ej_couplings(shapes[k], per, 1100 + i)[0]
        insts.append((J, per, None))
    beta = geometric_ladder(n_beta, 0.2, 3.0)
    n = max(int(np.prod(s)) for s in shapes)
    cycles = 33 if n <= 512 else 2
    ctx = sg.apt(insts, beta, SEED, reps_per_beta=reps)
    trace = ctx.run_apt(cycles, S, cutoff, record_every=1)
    assert ctx.launch_config() == 0   # no run in tiles
    ctx.sweep(S)
    spins, E, counts = ctx.spins(), ctx.energy(), ctx.swap_counts()
    if len(shapes) > 1:
        pick = list(range(16)) + [n_inst - 1]
    else:
        pick = range(0, n_inst, max(1, n_inst // (12 if n < 100 else 2)))
    for i in pick:
        lat = oracle.Lattice(*insts[i])
        sp = oracle.apt_init(lat, i, n_beta * reps, SEED)
        ctr, oE = np.zeros(3, np.uint32), np.zeros(n_beta * reps, np.int64)
        best = np.array([np.iinfo(np.int64).max], np.int64)
        rc, otr, oacc = oracle.apt_run(lat, i, beta, reps, SEED, cycles, S, cutoff, 1, ctr, sp, oE, best)
        assert rc == 0 and np.array_equal(trace[i], otr) and np.array_equal(counts[i], oacc), f"instance {i}"
        for k in range(S):
            oracle.apt_sweep(lat, i, np.repeat(beta, reps), SEED, cycles * S + k, sp)
        assert np.array_equal(spins[i, :, :lat.n], sp), f"spins, instance {i}"
        assert E[i].tolist() == [oracle.energy(lat, v) for v in sp], f"energies, instance {i}"


@pytest.mark.parametrize("shape,n_inst,n_chains", [((18, 18, 18), 270, 8), ((22, 22, 22), 3, 16)])
def test_adaptive_words_of_large_lattices(shape, n_inst, n_chains):
    """The adaptive kernel's wide bond counters (more than ten sites per thread), with 512 and 1024
    threads."""
    insts = [(ej_couplings(shape, 7, 1200 + i)[0], 7, None) for i in range(n_inst)]
    kw = dict(beta0=0.4, alpha=1.25, tol=0.01, n_chains=n_chains, sweeps=4, tail=3, max_steps=2)
    got = sg.adaptive_ladder(insts, 21, **kw)
    for i in {0, n_inst - 1}:
        beta, sigma = oracle.adaptive_ladder(oracle.Lattice(*insts[i]), i, 21, **kw)[:2]
        assert np.array_equal(got[i][0], beta) and np.array_equal(got[i][1], sigma), f"instance {i}"


def test_tuner_leaves_out_codes_that_are_the_same_kernel(tmp_path, monkeypatch):
    """Contexts whose work-groups have 512 or 1024 threads: codes 7..12 are codes 1..6."""
    monkeypatch.setenv("SG_TUNE_CACHE", str(tmp_path / "tune.txt"))
    for n_inst in range(1, 9):
        insts = [(ej_couplings((12, 12, 12), 7, 1300 + i)[0], 7, None) for i in range(n_inst)]
        ctx = sg.apt(insts, geometric_ladder(16, 0.2, 3.0), SEED, reps_per_beta=2)
        ctx.run_apt(2, 1, 1.0)
        assert ctx.launch_config() not in range(7, 13)


@pytest.mark.parametrize("shape,M,R,steps,launches", [((4, 3, 2), 6, 2, 129, 1), ((4, 3, 2), 6, 2, 256, 1),
                                                      ((4, 3, 2), 6, 2, 257, 2), ((4, 3, 2), 6, 2, 289, 3),
                                                      ((15, 15, 15), 4, 2500, 289, 2)])
def test_sqa_launches_of_a_schedule(shape, M, R, steps, launches):
    """A schedule of up to 256 steps is one launch (nothing to wait for); a longer one starts with a
    short launch unless its state is large (here 2500 x 27 KB)."""
    J, _ = ej_couplings(shape, 7, 521)
    ctx = sg.sqa([(J, 7, None)], M, R, 3.0, SEED)
    ctx.sqa_anneal(np.full(2, 1.0))   # the work-group size is settled
    ctx.kernel_timing(True)
    ctx.sqa_anneal(np.linspace(3.0, 0.1, steps))
    assert ctx.kernel_time()[1] == launches
