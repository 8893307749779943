"""GPU parity of the interaction passes' own rules: which pass a plan takes and how its items are cut.

The oracle is the reference (plain C, FP64); bar 1e-12, as for every FP64 potential.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import core  # noqa: E402
from paper_2012_06925_amd import _lib, inputs  # noqa: E402

PARITY = 1e-12


def _plan(p, targets=None, **kw):
    from paper_2012_06925_amd import api
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()        # noqa: E731
    t = None if targets is None else [dev(a) for a in (targets.x, targets.y, targets.z)]
    return api.Plan(t, [dev(a) for a in (p.x, p.y, p.z, p.q)], **kw)


def _computes(plan, n=2):
    return [plan.compute().cpu().numpy() for _ in range(n)]


def _close(got, ref):
    assert core.rel_l2(got, ref) < PARITY and core.max_rel(got, ref) < PARITY, (core.rel_l2(got, ref),
                                                                               core.max_rel(got, ref))


@pytest.mark.parametrize("kernel", ["yukawa", "oscillatory", "regcoulomb"])
@pytest.mark.parametrize("n,leaf,degree", [(5001, 40, 2), (9000, 300, 3), (6001, 700, 4)])
def test_symmetric_passes_of_the_other_kernels(kernel, n, leaf, degree):
    # leaves of one wave, of two per lane and of more than one tile; some
    # points twice (r = 0 inside a leaf and in the guarded ranges)
    p = inputs.particles(n, "uniform", seed=71)
    for a in (p.x, p.y, p.z):
        a[1:40:2] = a[0:39:2]
    plan = _plan(p, kernel=kernel, theta=0.8, degree=degree, leaf=leaf)
    a, b = _computes(plan)
    st = plan.stats()
    plan.close()
    assert st["pass_interactions"][2] > 0 and st["pass_interactions"][4] > 0
    assert np.array_equal(a, b)
    _close(a, core.bldtt(p, p, kernel=kernel, theta=0.8, degree=degree, leaf=leaf))


@pytest.mark.parametrize("kernel,param,shift", [("yukawa", -0.5, 0.0), ("yukawa", 1e101, 0.0), ("regcoulomb", 0.01, 2e17),
                                                ("yukawa", 0.5, 1e18)])
def test_padding_unsafe_problems_stay_one_sided(kernel, param, shift):
    # kernel values that grow with the distance or overflow at the padding,
    # and particles out where the padding sits, take the passes without padding
    p = inputs.particles(3000, "uniform", seed=72)
    if shift:
        for a in (p.x, p.y, p.z):
            a *= 1e16
            a += shift
    kw = dict(kernel=kernel, param=param, theta=0.7, degree=3, leaf=100)
    plan = _plan(p, **kw)
    got = _computes(plan, 1)[0]
    st = plan.stats()
    plan.close()
    assert st["pass_interactions"][2] == 0 and st["pass_interactions"][4] == 0
    one = _plan(p, flags=_lib.ONE_SIDED_PP, **kw)
    ref = _computes(one, 1)[0]
    one.close()
    assert np.all(np.isfinite(ref)) and np.array_equal(got, ref)


@pytest.mark.parametrize("kernel", ["coulomb", "yukawa", "oscillatory", "regcoulomb"])
@pytest.mark.parametrize("n,leaf,degree", [(6000, 50, 3), (9001, 120, 5), (12000, 300, 6)])
def test_mirrored_pc_cp_pairs_once_for_both(kernel, n, leaf, degree):
    # leaves smaller than the proxy grids: PC pairs and their CP mirrors, tiles
    # of one wave, of two and of four targets per lane
    p = inputs.particles(n, "gaussian", seed=73)
    kw = dict(kernel=kernel, theta=0.8, degree=degree, leaf=leaf)
    plan = _plan(p, **kw)
    a, b = _computes(plan)
    st, lists, tree = plan.stats(), plan.lists(), plan.tree()
    plan.close()
    one = _plan(p, flags=_lib.ONE_SIDED_PP, **kw)
    c = _computes(one, 1)[0]
    st1 = one.stats()
    one.close()
    assert st["n_entries"]["PC"] > 0 and st["interactions"] == st1["interactions"]
    # what the one-way particle pass keeps: PC pairs without a mirror, PP pairs
    # of which one side is no leaf or that are listed one way
    n, is_leaf, P = tree["count"], tree["nchild"] == 0, (degree + 1) ** 3
    pairs = {k: set(zip(*(v.tolist() for v in lists[k]))) for k in ("PP", "PC", "CP")}
    left = sum(int(n[a]) * P for a, b in pairs["PC"] if (b, a) not in pairs["CP"])
    left += sum(int(n[a]) * int(n[b]) for a, b in pairs["PP"]
                if a != b and not (is_leaf[a] and is_leaf[b] and (b, a) in pairs["PP"]))
    assert st["pass_interactions"][0] == left < st1["interactions"]["PC"] + st1["interactions"]["PP"]
    assert np.array_equal(a, b)
    ref = core.bldtt(p, p, **kw)
    _close(a, ref)
    _close(c, ref)


@pytest.mark.parametrize("leaf,degree", [(20, 3), (30, 4), (60, 5), (200, 6), (300, 7)])
def test_batch_pc_cp_pairs_tiled_over_the_grids(leaf, degree):
    # grids of 64 (one target per lane), 125 (two), 216 and 343 (four, a tail of
    # two), 512 (two full tiles), against clusters of fewer particles
    from paper_2012_06925_amd import api
    probs = [inputs.particles(n, "gaussian", seed=80 + k) for k, n in enumerate((900, 4001, 9000))]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()        # noqa: E731
    b = api.Batch([(None, [dev(a) for a in (p.x, p.y, p.z, p.q)]) for p in probs], kernel="coulomb", theta=0.8,
                  degree=degree, leaf=leaf)
    got = [[o.cpu().numpy() for o in b.compute()] for _ in range(2)]
    assert b.stats()["n_entries"]["PC"] > 0
    b.close()
    for p, x, y in zip(probs, *got):
        assert np.array_equal(x, y)
        _close(x, core.bldtt(p, p, kernel="coulomb", theta=0.8, degree=degree, leaf=leaf))


@pytest.mark.parametrize("kernel", ["coulomb", "yukawa", "oscillatory", "regcoulomb"])
@pytest.mark.parametrize("nsel", [1, 255, 257, 513, 1030])
def test_direct_sum_for_every_group_size(kernel, nsel):
    # one, two and four targets per work group, a last group that is not full,
    # fewer sources than threads, and every target against itself once
    from paper_2012_06925_amd import api
    for n in (nsel, 5003):
        p = inputs.particles(max(n, nsel), "uniform", seed=74)
        p.x[-1], p.y[-1], p.z[-1] = p.x[0], p.y[0], p.z[0]
        dev = [torch.from_numpy(a).cuda() for a in (p.x, p.y, p.z, p.q)]
        sel = np.sort(np.random.default_rng(3).choice(p.n, nsel, replace=False)).astype(np.int64)
        got = api.direct_sum(dev[:3], dev, kernel=kernel, sel=torch.from_numpy(sel).cuda()).cpu().numpy()
        ref = core.direct_sum(p, p, kernel=kernel)[sel]
        assert np.abs(got - ref).max() <= 1e-13 * max(np.abs(ref).max(), 1e-300)


@pytest.mark.parametrize("kernel,param", [("coulomb", None), ("yukawa", 0.5), ("yukawa", -0.5), ("regcoulomb", 0.005),
                                          ("regcoulomb", 1e160)])
def test_direct_sum_at_the_ends_of_the_range(kernel, param):
    # squared distances (and param^2) beyond the largest double give 1/inf = 0, not
    # inf * 0; points 1E-150 apart, whose squares are near the smallest double, count
    from paper_2012_06925_amd import api
    rng = np.random.default_rng(5)
    p = inputs.particles(700, "uniform", seed=75)
    p.x[:50], p.y[:50], p.z[:50] = 1e-150 * rng.random((3, 50))
    far = param is None or param > 0                       # exp(inf)/inf has no value
    if far:
        p.x[600:] = 1e200 * rng.choice([-3.0, -2.0, 1.0, 2.0], 100) + 1e198 * rng.random(100)
    dev = [torch.from_numpy(a).cuda() for a in (p.x, p.y, p.z, p.q)]
    got = api.direct_sum(dev[:3], dev, kernel=kernel, param=param).cpu().numpy()
    ref = core.direct_sum(p, p, kernel=kernel, param=param)
    p.q = np.abs(p.q)
    scale = core.direct_sum(p, p, kernel=kernel, param=param)      # each term to a few roundings
    assert np.all(np.isfinite(ref)) and np.all(np.isfinite(got))
    assert np.all(np.abs(got - ref) <= 1e-14 * scale), np.max(np.abs(got - ref) / np.maximum(scale, 1e-300))


@pytest.mark.parametrize("kernel,param,scale", [("yukawa", 0.0, 1.0), ("yukawa", 1e-3, 1.0), ("yukawa", 20.0, 1.0),
                                                ("yukawa", 300.0, 1.0), ("yukawa", 1000.0, 1.0), ("yukawa", -0.5, 1.0),
                                                ("regcoulomb", 3.0, 1.0), ("oscillatory", None, 60.0)])
def test_values_over_the_parameters_range(kernel, param, scale):
    # exponents from nothing to far below the smallest double (r up to 3.4), a
    # growing exponential, distances of up to 100 wavelengths: the symmetric
    # passes, the one-sided ones and the direct sum, each against the oracle
    from paper_2012_06925_amd import api
    p = inputs.particles(4001, "uniform", seed=76)
    for a in (p.x, p.y, p.z):
        a *= scale
    kw = dict(kernel=kernel, param=param, theta=0.7, degree=3, leaf=60)
    ref = core.bldtt(p, p, **kw)
    for flags in (0, _lib.ONE_SIDED_PP):
        plan = _plan(p, flags=flags, **kw)
        got = _computes(plan, 1)[0]
        plan.close()
        _close(got, ref)
    dev = [torch.from_numpy(a).cuda() for a in (p.x, p.y, p.z, p.q)]
    _close(api.direct_sum(dev[:3], dev, kernel=kernel, param=param).cpu().numpy(),
           core.direct_sum(p, p, kernel=kernel, param=param))


@pytest.mark.parametrize("param", [1e300, 1.2e308, 1.79e308])
def test_yukawa_with_a_param_near_the_largest_double(param):
    # param * log2(e) is infinite from 1.25E308 on; every value underflows to 0
    p = inputs.particles(3000, "uniform", seed=77)
    plan = _plan(p, kernel="yukawa", param=param, theta=0.7, degree=3, leaf=60)
    got = _computes(plan, 1)[0]
    plan.close()
    assert not np.any(got)


@pytest.mark.parametrize("n", [1, 63, 300, 8191, 8192])
@pytest.mark.parametrize("nsel", [1, 300, 1030])
def test_direct_sum_for_few_and_many_sources(n, nsel):
    # groups of 4 waves below 8192 sources and of 16 from there on, also with
    # fewer sources than threads, for one, two and four targets per group
    from paper_2012_06925_amd import api
    t, s = inputs.particles(nsel, "gaussian", seed=78), inputs.particles(n, "uniform", seed=79)
    dev = lambda *v: [torch.from_numpy(a).cuda() for a in v]                 # noqa: E731
    got = api.direct_sum(dev(t.x, t.y, t.z), dev(s.x, s.y, s.z, s.q)).cpu().numpy()
    ref = core.direct_sum(t, s)
    s.q = np.abs(s.q)
    assert np.all(np.abs(got - ref) <= 1e-14 * core.direct_sum(t, s))


@pytest.mark.parametrize("kernel", ["coulomb", "yukawa"])
def test_mirrored_pc_cp_pairs_in_tiles_of_several_slabs(kernel):
    # more than 8192 leaves: particle tiles of whole leaves of up to 600, in two and
    # four slabs of the work group, against grids of 1000 and the other way round
    p = inputs.particles(5_000_000, "gaussian", seed=96)
    kw = dict(kernel=kernel, theta=0.8, degree=9, leaf=600)
    phi = []
    for flags in (0, _lib.ONE_SIDED_PP):
        plan = _plan(p, flags=flags | _lib.DEVICE_TREE, **kw)
        phi += _computes(plan, 2 - (flags != 0))
        n, st = plan.tree()["count"], plan.stats()
        lists = plan.lists()["PC"]
        plan.close()
    assert np.array_equal(phi[0], phi[1])
    assert st["n_entries"]["PC"] > 0 and np.any(n[lists[0]] > 256)
    _close(phi[0], phi[2])


def test_particles_beyond_the_padding_against_the_oracle():
    # 2E17 away, where coordinates are 32 apart: proxy points of boxes of 1E15 round to
    # 3e-14 of their size, which 3000 charges of both signs may bring to 1e-12 and more
    p = inputs.particles(3000, "uniform", seed=72)
    for a in (p.x, p.y, p.z):
        a *= 1e16
        a += 2e17
    kw = dict(kernel="regcoulomb", param=0.01, theta=0.7, degree=3, leaf=100)
    plan = _plan(p, **kw)
    got = _computes(plan, 1)[0]
    plan.close()
    ref = core.bldtt(p, p, **kw)
    assert core.rel_l2(got, ref) < 1e-10 and core.max_rel(got, ref) < 1e-10
