"""The one-pass chemistry kernel (persistent lanes that take the next cell
as soon as theirs has filled dt_RT, long chains of the previous pass first)
against the two-pass chemistry (a lockstep head pass, then the queued cells
in a persistent tail): the same bits in every field and the same counters,
for both precisions, one to three groups, smoothed RT and the case without
the on-the-spot approximation, over several steps of the split rt_step and
for rt_thermochem alone; with non-finite cells; with a list of long chains
larger than the room it has; and on a grid large enough (over the 131,072
lanes of the first fill) that most cells reach their lane as a refill.  The
order and the lists are in use above 131,072 cells, one per lane of the first
fill; the smaller grids here take their cells in grid order."""
import numpy as np
import pytest
import torch

import rt_inputs as ri
from test_gpu_parity import chem_compare, gas, make_pair, random_rad

pytestmark = pytest.mark.gpu

FIELDS = ("N", "F", "xHII", "xHeII", "xHeIII", "T", "nacc", "natt")
COUNTS = ("substeps_total", "attempts_total", "attempts_max", "flags", "substep_hist")


def compare(a, b):
    ga, gb = a.state_numpy(), b.state_numpy()
    for k in FIELDS:
        assert np.array_equal(ga[k], gb[k], equal_nan=True), k
    sa, sb = a.stats(), b.stats()
    for k in COUNTS:
        assert sa[k] == sb[k], (k, sa[k], sb[k])
    for k in ("injected", "absorbed", "outflow", "photons"):
        assert np.array_equal(sa[k], sb[k], equal_nan=True), k
    return sa


def lognormal_pair(n, fp32, nH_mean, smooth=False, otsa=True, steps=4, spectrum=None, queue_cap=None):
    from paper_1304_7126_amd import RTContext
    w = ri.lognormal_box(n, 6.6 * n / 128, 6, steps=steps, seed=5, spectrum=spectrum)
    w.nH_mean = nH_mean
    w.otsa = otsa
    ijk, nd = ri.random_sources(w.n, w.n_sources, w.seed)
    ctxs = []
    for path in ("two-pass", "one-pass"):
        c = RTContext.for_workload(w, fp32=fp32, counters=True, smooth=smooth, N_floor=1e-12 if smooth else 0.0)
        c.load_state(ri.initial_state(w))
        c.set_sources(ijk, c.source_rates(nd))
        c.set_transport_path("zmarch")
        c.set_chem_path(path)
        c.set_accounting(True)
        if queue_cap is not None:
            c.set_tuning(-1, queue_cap)
        c.reset_stats()
        ctxs.append(c)
    return w, ctxs


@pytest.mark.parametrize("fp32", [True, False])
@pytest.mark.parametrize("M", [1, 2, 3])
def test_one_pass_equals_two_pass_step(fp32, M):
    spec = ri.Spectrum(kind="bb", T_bb=1e5, edges_eV={1: ri.EDGES_1, 2: ri.EDGES_2, 3: ri.EDGES_3}[M])
    # dense gas: I-front cells take tens to hundreds of attempts, so the
    # list of long chains is in use from the second step on
    w, (a, b) = lognormal_pair(24, fp32, 0.1, spectrum=spec, steps=6)
    dt = a.courant_dt()
    for _ in range(w.steps):
        a.step(dt, 1)
        b.step(dt, 1)
    s = compare(a, b)
    print(f"# one-pass vs two-pass M={M} fp32={fp32}: attempts max {s['attempts_max']}", flush=True)
    assert s["attempts_max"] >= 48


@pytest.mark.parametrize("smooth,otsa", [(True, True), (False, False), (True, False)])
def test_one_pass_equals_two_pass_variants(smooth, otsa):
    w, (a, b) = lognormal_pair(20, True, 0.03, smooth=smooth, otsa=otsa, steps=5)
    dt = a.courant_dt()
    for _ in range(w.steps):
        a.step(dt, 1)
        b.step(dt, 1)
    compare(a, b)


def test_one_pass_with_a_list_larger_than_its_room():
    # a queue of 7 cells: most long chains are not listed and go through
    # the sweep over all cells like any other
    w, (a, b) = lognormal_pair(24, True, 0.1, steps=6, queue_cap=7)
    dt = a.courant_dt()
    for _ in range(w.steps):
        a.step(dt, 1)
        b.step(dt, 1)
    s = compare(a, b)
    assert s["attempts_max"] >= 48


@pytest.mark.parametrize("fp32", [True, False])
def test_one_pass_thermochem_alone_with_a_nonfinite_cell(fp32):
    rng = np.random.default_rng(3)
    n = (37, 21, 19)
    N, F = random_rad(n, 3, rng)
    st = {"N": N, "F": F, **gas(n, rng)}
    st["T"][4, 5, 6] = np.nan
    st["N"][1, 7, 3, 2] = np.inf
    # a cell whose flux alone is not finite (the one-pass kernel finds it
    # only when it writes the cell)
    st["F"][2, 1, 10, 11, 12] = np.nan
    ctxs = []
    for path in ("two-pass", "one-pass"):
        c, _ = make_pair(n, (0,) * 6, 3, 1, fp32=fp32)
        c.load_state(st)
        c.set_chem_path(path)
        c.set_accounting(True)
        c.reset_stats()
        ctxs.append(c)
    dt = ctxs[0].courant_dt()
    for c in ctxs:
        for _ in range(3):
            c.thermochem(dt)
    s = compare(*ctxs)
    assert s["flags"] & 2


@pytest.mark.parametrize("fp32", [True, False])
def test_one_pass_refills_on_a_large_grid(fp32):
    # 96^3 cells: 3.4x the lanes of the first fill, so that most cells are
    # taken by lanes whose previous cell is done
    w, (a, b) = lognormal_pair(96, fp32, 0.03, steps=3)
    for c in (a, b):
        st = c.state_numpy()
        st["nH"] = c.nH.cpu().numpy()
        # non-finite inputs late in the grid: a flux, a density, a temperature
        st["F"][1, 2, 90, 91, 92] = np.nan
        st["N"][0, 80, 3, 4] = np.inf
        st["T"][70, 60, 50] = np.nan
        c.load_state(st)
    dt = a.courant_dt()
    for _ in range(w.steps):
        a.step(dt, 1)
        b.step(dt, 1)
    s = compare(a, b)
    assert s["flags"] & 2


@pytest.mark.parametrize("lo,hi", [(-2.0, 0.5), (0.9, 1.3), (7.2, 7.8), (7.5, 10.0)])
def test_one_pass_at_the_ends_of_the_lds_rate_table(lo, hi):
    # 10^lo .. 10^hi K: below, across and above the octaves (2^-3 K .. 2^25 K,
    # the HeIII fits at a quarter) whose rates the persistent kernels read from
    # LDS; the head pass reads all from global memory, so the bits must agree,
    # and the oracle evaluates the formulas
    rng = np.random.default_rng(int(10 * (hi + 20)))
    n = (24, 17, 9)
    N, F = random_rad(n, 3, rng)
    gs = gas(n, rng)
    gs["T"] = 10 ** rng.uniform(lo, hi, gs["T"].shape)
    st = {"N": 1e-3 * N, "F": 1e-3 * F, **gs}
    ctxs = []
    for path in ("two-pass", "one-pass"):
        ctx, o = make_pair(n, (0,) * 6, 3, 0)
        ctx.set_chem_path(path)
        ctx.load_state(st)
        ctx.thermochem(ctx.courant_dt())
        ctxs.append(ctx)
    compare(*ctxs)
    fl, nacc, natt = o.thermochem(st, ctxs[0].courant_dt(), want_counts=True)
    st["nacc"], st["natt"] = nacc, natt
    chem_compare(ctxs[1].state_numpy(), st)


@pytest.mark.parametrize("n,fp32,smooth,otsa,cap", [
    (50, True, False, True, None),    # 125,000 cells: one per lane, in grid order
    (51, True, False, True, None),    # 132,651: ordered, the last piece of 1,579 cells
    (51, False, False, True, None),
    (51, True, True, True, None),
    (51, False, False, False, None),
    (64, True, False, True, 0),       # 64 pieces, eight to a slab; a queue the two passes do not have
])
def test_one_pass_in_sorted_pieces(n, fp32, smooth, otsa, cap):
    # a state just set (warm gas listed), then counts of earlier steps and
    # chains of 48 attempts and more on the lists
    w, (a, b) = lognormal_pair(n, fp32, 0.1, smooth=smooth, otsa=otsa, steps=4, queue_cap=cap)
    dt = a.courant_dt()
    for _ in range(w.steps):
        a.step(dt, 1)
        b.step(dt, 1)
    s = compare(a, b)
    assert s["attempts_max"] >= 48


@pytest.mark.parametrize("smooth,otsa", [(False, True), (False, False), (True, True)])
@pytest.mark.parametrize("path", ["one-pass", "two-pass", "cell"])
def test_isothermal_cells_without_a_positive_temperature(path, smooth, otsa):
    # no rate is defined at T <= 0: such a cell fails every attempt, keeps its
    # state and raises the cap flag; the other cells are as without it
    n = (21, 7, 3)
    rng = np.random.default_rng(11)
    N, F = random_rad(n, 3, rng)
    st = {"N": 1e-3 * N, "F": 1e-3 * F, **gas(n, rng)}
    for k, v in enumerate((0.0, -0.0, -1e4, -1e-300, -1e300)):
        st["T"][k % 3, 1 + k, 4 * k] = v
    st["T"][2, 6, 20] = 0.0
    bad = ~(st["T"] > 0)
    ctx, o = make_pair(n, (0,) * 6, 3, 0, isothermal=True, smooth=smooth, otsa=otsa, N_floor=1e-12 if smooth else 0.0)
    ctx.set_transport_path("cell" if path == "cell" else "zmarch")
    ctx.set_chem_path("auto" if path == "cell" else path)
    ref, _ = make_pair(n, (0,) * 6, 3, 0, isothermal=True, smooth=smooth, otsa=otsa, N_floor=1e-12 if smooth else 0.0)
    ok = {**st, "T": np.where(bad, 1e4, st["T"])}
    for c, s in ((ctx, st), (ref, ok)):
        c.load_state(s)
        c.reset_stats()
        c.step(c.courant_dt(), 1)
    g, r = ctx.state_numpy(), ref.state_numpy()
    for k in ("xHII", "xHeII", "xHeIII", "T"):
        assert np.array_equal(g[k][bad], st[k][bad]), k
    assert np.all(g["nacc"][bad] == 0) and np.all(g["natt"][bad] == 100000)
    for k in FIELDS:
        m = np.broadcast_to(~bad, g[k].shape)
        assert np.array_equal(g[k][m], r[k][m]), k
    s = ctx.stats()
    assert s["flags"] == ref.stats()["flags"] | 1 and s["attempts_max"] == 100000
    assert not ref.stats()["flags"] & 1


def test_isothermal_batch_box_without_a_positive_temperature():
    from paper_1304_7126_amd.batch import batch_from_specs
    specs = [ri.BoxSpec(side=9, M=1, nH=1e-2, n_sources=1, seed=5), ri.BoxSpec(side=5, M=3, nH=1e-2, n_sources=1, seed=6)]
    b, ws, srcs = batch_from_specs(specs, 6.6 * ri.KPC / 128, isothermal=True)
    b.boxes[1].T[1, 2, 3] = 0.0
    b.boxes[1].T[4, 4, 4] = -3.0
    x0 = b.boxes[1].xHII.clone()
    b.reset_stats()
    b.step(b.courant_dt(), 1)
    b.synchronize()
    s = b.stats()
    assert s["flags"] == 1 and s["attempts_max"] == 100000
    assert torch.equal(b.boxes[1].xHII[1, 2, 3], x0[1, 2, 3]) and torch.equal(b.boxes[1].xHII[4, 4, 4], x0[4, 4, 4])


@pytest.mark.parametrize("isothermal", [True, False])
def test_temperatures_far_below_the_lds_rate_table(isothermal):
    # 1e-18 to 1e-10 K mean nothing, but they are accepted and the oracle
    # evaluates the formulas there (without OTSA such gas reaches the attempt
    # cap on either side, at a count that rounding decides)
    rng = np.random.default_rng(23)
    n = (11, 5, 3)
    N, F = random_rad(n, 3, rng)
    gs = gas(n, rng)
    gs["xHII"] = rng.uniform(0.05, 0.9, gs["T"].shape)
    gs["T"] = 10 ** rng.uniform(-18, -10, gs["T"].shape)
    st = {"N": 1e-3 * N, "F": 1e-3 * F, **gs}
    ctxs = []
    for path in ("two-pass", "one-pass"):
        ctx, o = make_pair(n, (0,) * 6, 3, 0, isothermal=isothermal)
        ctx.set_chem_path(path)
        ctx.load_state(st)
        ctx.thermochem(ctx.courant_dt())
        ctxs.append(ctx)
    compare(*ctxs)
    fl, nacc, natt = o.thermochem(st, ctxs[0].courant_dt(), want_counts=True)
    st["nacc"], st["natt"] = nacc, natt
    chem_compare(ctxs[1].state_numpy(), st)


def test_attempt_counts_beyond_32_bits_per_lane():
    # every cell at the cap of INT_MAX attempts (T = 0 held), more than two
    # cells per persistent lane: the total is exact
    from paper_1304_7126_amd import RTContext
    w = ri.lognormal_box(96, 6.6 * 96 / 128, 1, steps=1, seed=1)
    cap = 2 ** 31 - 1
    c = RTContext.for_workload(w, fp32=True, isothermal=True, max_attempts=cap)
    c.load_state(ri.initial_state(w))
    c.T.zero_()
    for k in range(2):
        c.reset_stats()
        c.thermochem(c.courant_dt())
        s = c.stats()
        assert s["attempts_total"] == 96 ** 3 * cap and s["attempts_max"] == cap and s["substeps_total"] == 0
        assert s["flags"] == 1


def warm_state(w, frac, seed):
    """A restart: frac of the cells ionised and warm, scattered in the first
    half of the grid's planes and as one block in the rest."""
    rng = np.random.default_rng(seed)
    st = ri.initial_state(w)
    sh = st["T"].shape
    m = rng.uniform(size=sh) < frac
    m[sh[0] // 2:] = False
    m[sh[0] // 2: sh[0] // 2 + int(frac * (sh[0] - sh[0] // 2))] = True
    st["T"][m] = 10 ** rng.uniform(3.8, 4.4, m.sum())
    st["xHII"][m] = 0.99
    st["xHeII"][m] = 0.9
    st["N"] = np.where(m, 1e-5 * np.array([1.0, 0.5, 0.1]).reshape(3, 1, 1, 1), st["N"])
    return st


@pytest.mark.parametrize("frac", [1.0, 0.26, 0.24, 0.02])
@pytest.mark.parametrize("fp32,smooth", [(True, False), (False, False), (True, True)])
def test_first_pass_of_a_warm_state(fp32, smooth, frac):
    # a state without counts above the lanes of the first fill: warm cells go
    # to the lists where they are a quarter of their piece or less
    w, (a, b) = lognormal_pair(52, fp32, 1e-3, smooth=smooth, steps=2)
    st = warm_state(w, frac, 7)
    dt = a.courant_dt()
    for c in (a, b):
        c.load_state(st)
        c._bind()
        c.set_accounting(True)
        c.step(dt, 2)
    compare(a, b)


def test_first_pass_of_a_warm_state_costs_no_more_than_the_next():
    # (all warm cells of a state without counts on the lists: 2.9 times)
    w = ri.lognormal_box(192, 13.2 * 192 / 256, 1, steps=1, seed=2)
    from paper_1304_7126_amd import RTContext
    c = RTContext.for_workload(w, fp32=True)
    c.load_state(warm_state(w, 1.0, 3))
    keep = [t.clone() for t in (c.N, c.F, c.xHII, c.xHeII, c.xHeIII, c.T)]
    dt = c.courant_dt()
    ms = {0: [], 1: []}
    for _ in range(6):
        for t, k in zip((c.N, c.F, c.xHII, c.xHeII, c.xHeIII, c.T), keep):
            t.copy_(k)
        c._bind()
        for p in (0, 1):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda.synchronize()
            e0.record()
            c.thermochem(dt)
            e1.record()
            torch.cuda.synchronize()
            ms[p].append(e0.elapsed_time(e1))
    print(f"# first pass {min(ms[0]):.3f} ms, second {min(ms[1]):.3f} ms", flush=True)
    assert min(ms[0]) < 1.8 * min(ms[1])


@pytest.mark.parametrize("M,fp32,iso,smooth,otsa,cap", [
    (1, True, False, False, True, None), (2, False, False, False, True, None), (1, False, True, False, True, None),
    (3, True, True, False, True, None), (2, True, False, True, False, None), (3, False, False, True, False, 7)])
def test_sorted_pieces_of_every_variant(M, fp32, iso, smooth, otsa, cap):
    # 53 x 51 x 50 = 135,150 cells: ordered, with lists from the second step on
    # (gas of one class when it is isothermal), against the two passes
    from paper_1304_7126_amd import RTContext
    w = ri.lognormal_box(53, 6.6 * 53 / 128, 6, steps=4, seed=9,
                         spectrum=ri.Spectrum(kind="bb", T_bb=1e5, edges_eV={1: ri.EDGES_1, 2: ri.EDGES_2, 3: ri.EDGES_3}[M]))
    w.nH_mean, w.otsa = 0.1, otsa
    st = ri.initial_state(w)
    w.n = (53, 51, 50)
    st = {k: np.ascontiguousarray(v[..., :50, :51, :]) for k, v in st.items()}
    if iso:
        st["T"][:] = 1e4
    ijk, nd = ri.random_sources(w.n, w.n_sources, w.seed)
    ctxs = []
    for path in ("two-pass", "one-pass"):
        c = RTContext.for_workload(w, fp32=fp32, counters=True, smooth=smooth, isothermal=iso, N_floor=1e-12 if smooth else 0.0)
        c.load_state(st)
        c.set_sources(ijk, c.source_rates(nd))
        c.set_chem_path(path)
        c.set_accounting(True)
        if cap is not None:
            c.set_tuning(-1, cap)
        c.reset_stats()
        c.step(c.courant_dt(), w.steps)
        ctxs.append(c)
    s = compare(*ctxs)
    listed = int((ctxs[1].natt >= 20).sum())
    print(f"# M={M} fp32={fp32} iso={iso} smooth={smooth} otsa={otsa}: {listed} cells of 20 attempts or more", flush=True)
    assert listed > 0 and s["attempts_max"] >= 20


@pytest.mark.parametrize("lo,hi", [(-2.0, 0.5), (0.9, 1.3), (7.2, 7.8), (7.5, 10.0)])
def test_case_a_at_the_ends_of_the_lds_rate_table(lo, hi):
    # the emission's difference of two rates and the case A cooling from global
    # memory in lanes outside the LDS copy: one pass (LDS) and two passes (the
    # head pass reads all from global memory) bit for bit; the oracle where the
    # substeps do not end at the cap (cold gas without OTSA does)
    rng = np.random.default_rng(int(10 * (hi + 20)))
    n = (24, 17, 9)
    N, F = random_rad(n, 3, rng)
    gs = gas(n, rng)
    gs["T"] = 10 ** rng.uniform(lo, hi, gs["T"].shape)
    st = {"N": 1e-3 * N, "F": 1e-3 * F, **gs}
    ctxs = []
    for path in ("two-pass", "one-pass"):
        ctx, o = make_pair(n, (0,) * 6, 3, 0, otsa=False)
        ctx.set_chem_path(path)
        ctx.load_state(st)
        ctx.thermochem(ctx.courant_dt())
        ctxs.append(ctx)
    compare(*ctxs)
    if lo < 7.0:
        return
    fl, nacc, natt = o.thermochem(st, ctxs[0].courant_dt(), want_counts=True)
    st["nacc"], st["natt"] = nacc, natt
    chem_compare(ctxs[1].state_numpy(), st)
