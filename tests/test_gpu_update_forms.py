"""The update past its register form: one launch where one workgroup per joint is
the shorter path, two for more points, with the same bits (marked gpu)."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs
from tests.gpu_launches import launches

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GOAL = [1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4, 0.1, 0.45]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_13542_amd import storm

    storm.lib()


def _problem(n, h, beta=1.0, cov=0):
    pr = inputs.config1(5)
    p = pr.params
    p.n_particles, p.horizon, p.dt, p.beta, p.cov_per_step, p.n_null = n, h, np.full(h, 0.02), beta, cov, 3
    return pr


# 90000 points are the last that one workgroup per joint takes, 8192 particles the
# most; the register form ends at 512, 1088 and 2048 particles at 64, 30 and 1 steps
@pytest.mark.parametrize("n,h,count", [(512, 64, 1), (513, 64, 1), (1406, 64, 1), (1407, 64, 2), (1089, 30, 1),
                                       (3000, 30, 1), (3001, 30, 2), (2049, 1, 1), (8192, 10, 1), (8193, 10, 2)])
def test_launches_of_an_update(n, h, count):
    from paper_2104_13542_amd import storm

    goal = torch.tensor(GOAL, dtype=torch.float32, device="cuda")
    r = storm.Rollout(_problem(n, h))
    try:
        r.step(goal)
        assert len(launches(lambda: r.update(want_mean=False))) == count
    finally:
        r.close()


# a batch takes one workgroup per joint up to 8192 particles: the same problem on
# either side of the plain form's line, by the list and by all particles
@pytest.mark.parametrize("n,h,beta,cov", [(1407, 64, 1e-3, 0), (1407, 64, 1e6, 1), (3001, 30, 50.0, 0),
                                          (3000, 30, 1.0, 1), (8192, 11, 1e6, 0), (8192, 12, 0.5, 1),
                                          (4097, 22, 1e6, 0), (4096, 23, 1e6, 1), (8191, 64, 20.0, 1)])
def test_one_workgroup_per_joint_equals_chains(n, h, beta, cov):
    from paper_2104_13542_amd import storm

    goals = torch.tensor([GOAL, GOAL], dtype=torch.float32, device="cuda")
    probs = [_problem(n, h, beta, cov), _problem(40, 7)]
    b, r = storm.Batch(probs), storm.Rollout(probs[0])
    try:
        for _ in range(2):
            b.step(goals)
            r.step(goals[0])
            cmd, plain = b.update(shift=True), r.update(shift=True)[0]
            torch.cuda.synchronize()
            assert torch.equal(cmd[0], plain)
            for x, y in zip(b.get_state(0), r.get_state()):
                np.testing.assert_array_equal(x, y)
    finally:
        b.close()
        r.close()


def test_a_batch_holds_no_partial_sums_that_it_does_not_use():
    """Contexts of 2049 x 64 hold the chains' partial sums (448 KiB); a batch updates
    such problems with one workgroup per joint."""
    from paper_2104_13542_amd import storm

    def held(make):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        owned = make()
        torch.cuda.synchronize()
        used = free - torch.cuda.mem_get_info()[0]
        for o in owned:
            o.close()
        return used

    probs = [_problem(2049, 64) for _ in range(64)]
    storm.Rollout(_problem(8, 8)).close()
    batch = held(lambda: [storm.Batch(probs)])
    plain = held(lambda: [storm.Rollout(pr) for pr in probs])
    assert plain - batch >= 0.9 * 64 * 448 * 1024


# one workgroup per joint, then chains
@pytest.mark.parametrize("n,h", [(8192, 8), (8193, 8), (3001, 30)])
@pytest.mark.parametrize("which", ["first", "middle", "last"])
def test_a_cost_that_is_not_finite_keeps_the_policy(n, h, which):
    from paper_2104_13542_amd import storm

    pr = _problem(n, h)
    pr.params.n_null = 0
    eps = inputs.standard_normal(3, (7, n, h))
    eps[2, {"first": 0, "middle": n // 2, "last": n - 1}[which], h // 2] = np.inf
    goal = torch.tensor(GOAL, dtype=torch.float32, device="cuda")
    r = storm.Rollout(pr)
    try:
        before = r.get_state()
        r.step(goal, noise=torch.tensor(eps, dtype=torch.float32, device="cuda"))
        _, mean, sig = r.update(shift=False)
        torch.cuda.synchronize()
        after = r.get_state()
        assert r.status() == storm.FLAG_NONFINITE_COST
        np.testing.assert_array_equal(mean.cpu().numpy(), before[0])
        np.testing.assert_array_equal(sig.cpu().numpy(), before[1])
        np.testing.assert_array_equal(after[0], before[0])
        assert after[2] == before[2] + 1
    finally:
        r.close()
