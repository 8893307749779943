"""bldtt_set_allocator through the C ABI: plans and batches take their device
memory from the registered allocator and give all of it back; an allocator
that returns NULL makes the call fail with BLDTT_ENOMEM, every buffer
allocated before the failure released (counted in the callbacks)."""
import gc

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import core  # noqa: E402
from paper_2012_06925_amd import inputs  # noqa: E402


def _api():
    from paper_2012_06925_amd import api
    return api


class Counting:
    """Device memory from torch's caching allocator, counted; NULL after `fail_after` allocations."""

    def __init__(self, fail_after=None):
        self.fail_after = fail_after
        self.live = {}
        self.n_alloc = self.n_release = self.n_refused = 0

    def alloc(self, n):
        if self.fail_after is not None and self.n_alloc >= self.fail_after:
            self.n_refused += 1
            return 0
        p = torch.cuda.caching_allocator_alloc(n)
        self.live[p] = n
        self.n_alloc += 1
        return p

    def release(self, p):
        assert p in self.live, "released a pointer the allocator did not hand out"
        del self.live[p]
        self.n_release += 1
        torch.cuda.caching_allocator_delete(p)


def _src(n, seed):
    p = inputs.particles(n, "uniform", seed=seed)
    return p, [torch.from_numpy(a).cuda() for a in (p.x, p.y, p.z, p.q)]


def test_plan_memory_comes_from_the_registered_allocator():
    api = _api()
    p, src = _src(20_000, 90)
    cnt = Counting()
    api.set_allocator(cnt.alloc, cnt.release)
    try:
        plan = api.Plan(None, src, theta=0.7, degree=5, leaf=200)
        phi = plan.compute().cpu().numpy()
        phi2 = plan.compute().cpu().numpy()
        assert cnt.n_alloc > 10 and cnt.live
        plan.close()
        assert not cnt.live and cnt.n_release == cnt.n_alloc
    finally:
        api.use_torch_allocator()
    ref = core.bldtt(p, p, theta=0.7, degree=5, leaf=200)
    for got in (phi, phi2):
        assert core.rel_l2(got, ref) < 1e-12 and core.max_rel(got, ref) < 1e-12


def test_failing_allocator_gives_enomem_and_releases_everything():
    # count the allocations of a full setup, then refuse the first, the
    # second, one in the middle and the last of them
    api = _api()
    from paper_2012_06925_amd import _lib
    _, src = _src(30_000, 91)
    flags = _lib.FP32_EVAL | _lib.LEARNED_DEGREE
    kw = dict(theta=0.7, degree=5, leaf=200, flags=flags)
    probe = Counting()
    api.set_allocator(probe.alloc, probe.release)
    try:
        api.Plan(None, src, **kw).close()
    finally:
        api.use_torch_allocator()
    n = probe.n_alloc
    assert n > 8 and not probe.live
    for fail_after in sorted({0, 1, n // 2, n - 1}):
        gc.collect()
        torch.cuda.synchronize()
        base = torch.cuda.memory_allocated()
        cnt = Counting(fail_after)
        api.set_allocator(cnt.alloc, cnt.release)
        try:
            with pytest.raises(_lib.BldttError) as e:
                api.Plan(None, src, **kw)
        finally:
            api.use_torch_allocator()
        assert e.value.code == _lib.ENOMEM, e.value
        assert cnt.n_refused == 1 and cnt.n_alloc == fail_after, (fail_after, cnt.n_refused, cnt.n_alloc)
        assert not cnt.live and cnt.n_release == cnt.n_alloc
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated() <= base          # nothing the failed call took is still held


def test_failing_allocator_during_compute_and_batch_setup():
    # a plan set up normally whose allocator then refuses: the compute that
    # needs new buffers fails with ENOMEM, and destroying the plan releases all
    api = _api()
    from paper_2012_06925_amd import _lib
    _, src = _src(30_000, 92)
    cnt = Counting()
    api.set_allocator(cnt.alloc, cnt.release)
    try:
        plan = api.Plan(None, src, theta=0.7, degree=5, leaf=200)
        cnt.fail_after = cnt.n_alloc          # setup done: refuse every later request
        with pytest.raises(_lib.BldttError) as e:
            plan.compute()
        assert e.value.code == _lib.ENOMEM
        plan.close()
        assert not cnt.live and cnt.n_release == cnt.n_alloc
        # a batch whose setup runs out part way
        probs = [(None, tuple(torch.from_numpy(a).cuda() for a in (q.x, q.y, q.z, q.q)))
                 for _, q in inputs.batch_problems(count=6, seed=93, lo_exp=2.5, hi_exp=3.5)]
        cnt2 = Counting(fail_after=12)
        api.set_allocator(cnt2.alloc, cnt2.release)
        with pytest.raises(_lib.BldttError) as e:
            api.Batch(probs, theta=0.7, degree=5, leaf=60)
        assert e.value.code == _lib.ENOMEM
        assert not cnt2.live and cnt2.n_release == cnt2.n_alloc == 12
    finally:
        api.use_torch_allocator()


class RefuseOne(Counting):
    """Refuses one allocation only, the k-th."""

    def __init__(self, k):
        super().__init__()
        self.k = k

    def alloc(self, n):
        if self.n_alloc == self.k and self.n_refused == 0:
            self.n_refused = 1
            return 0
        return super().alloc(n)


@pytest.mark.parametrize("form", ["coulomb", "yukawa", "treecode", "tuned", "batch"])
def test_memory_that_only_saves_time_is_not_needed(form):
    # every allocation of a setup and a compute refused in turn: the call fails with
    # ENOMEM and releases all, or the plan goes on without and the results are right;
    # slots (yukawa: of the self pairs, at setup, and of the passes) are of that kind
    api = _api()
    from paper_2012_06925_amd import _lib, train_degree_model
    kw = dict(theta=0.8, degree=4, leaf=60)
    p, src = _src(4000, 94)
    tgt = None
    if form == "yukawa":
        kw["kernel"] = "yukawa"
    if form == "treecode":
        t = inputs.particles(300, "gaussian", seed=95, charges=False)
        tgt = [torch.from_numpy(a).cuda() for a in (t.x, t.y, t.z)]
        kw["flags"] = _lib.BLTC
    if form == "tuned":
        kw["flags"] = _lib.FP32_EVAL | _lib.LEARNED_DEGREE

    def run():
        if form == "batch":
            b = api.Batch([(None, src)], **kw)
            try:
                return b.compute()[0].cpu().numpy()
            finally:
                b.close()
        plan = api.Plan(tgt, src, **kw)
        try:
            if form == "tuned":
                plan.set_degree_model(train_degree_model.load_model(), fallback=4)
            a = plan.compute().cpu().numpy()
            assert (plan.compute().cpu().numpy() == a).all()
            return a
        finally:
            plan.close()

    probe = Counting()
    api.set_allocator(probe.alloc, probe.release)
    try:
        ref = run()
        assert probe.n_alloc > 10 and not probe.live
        went_on = 0
        for k in range(probe.n_alloc):
            one = RefuseOne(k)
            api.set_allocator(one.alloc, one.release)
            try:
                got = run()
            except _lib.BldttError as e:
                assert e.code == _lib.ENOMEM, (k, e)
            else:
                went_on += one.n_refused
                assert core.rel_l2(got, ref) < (1e-6 if form == "tuned" else 1e-12), k
            assert not one.live and one.n_release == one.n_alloc, k
    finally:
        api.use_torch_allocator()
    assert went_on >= {"yukawa": 3, "batch": 2}.get(form, 1), went_on
