"""The policy update of more particles than one workgroup per joint holds in
registers, in one workgroup per joint (up to 8192) and in parallel chains, against
the oracle's update fed with the kernel's own costs and controls, at the edges of
its forms and rows, for weights from one-hot to uniform, and with a cost that is
not finite (marked gpu)."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs
from tests.gpu_common import TOL_MEAN, f32, to_nhj

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_13542_amd import storm

    storm.lib()


def _problem(n, h, beta, cov):
    prob = inputs.config1(5)
    p = prob.params
    p.n_particles, p.horizon, p.dt, p.beta, p.cov_per_step, p.n_null = n, h, np.full(h, 0.02), beta, cov, 3
    prob.q0 = f32(prob.q0)
    return prob


# the register path holds 32 * (1024 // h) particles, and 2048 at most; the list
# 4096 weights; chains begin at 8193 particles
@pytest.mark.parametrize("n,h,beta,cov", [(2049, 1, 1.0, 0), (2049, 16, 1e-4, 1), (513, 64, 50.0, 0),
                                          (1089, 30, 1e6, 1), (545, 63, 1.0, 0), (32768, 3, 20.0, 0),
                                          (32769, 2, 1e6, 1), (70001, 5, 5.0, 0), (4097, 8, 1e6, 0),
                                          (8192, 8, 1e6, 1), (8193, 8, 1e6, 0)])
def test_split_update_against_oracle(oracle_lib, n, h, beta, cov):
    from paper_2104_13542_amd import storm

    prob = _problem(n, h, beta, cov)
    p = prob.params
    o = oracle_lib.Oracle(prob)
    goal = torch.tensor(f32(o.goal), dtype=torch.float32, device="cuda")
    rng = np.random.default_rng(n)
    mean0 = f32(rng.normal(0.0, 0.1, (h, 7)))
    s2 = f32(rng.uniform(0.005, 0.02, (h, 7) if cov else 7))
    r = storm.Rollout(prob)
    try:
        r.set_state(mean=mean0, sigma2=s2)
        out = r.step(goal, debug=True)
        cmd, mean, sig = r.update(shift=True)
        torch.cuda.synchronize()
        C, u = out["C"].cpu().double().numpy(), to_nhj(out["u"])
        got = [x.cpu().double().numpy() for x in (mean, sig, cmd)]
        state = r.get_state()
        assert r.status() == 0
    finally:
        r.close()
    up = o.update(C, u, mean0, s2)
    assert np.max(np.abs(got[0] - up["mean"])) <= TOL_MEAN
    assert np.max(np.abs(got[1] - up["sigma2"])) <= TOL_MEAN
    np.testing.assert_array_equal(got[2], got[0][0])
    assert state[2] == 1
    np.testing.assert_array_equal(state[0][:-1], mean.cpu().numpy()[1:])
    np.testing.assert_array_equal(state[0][-1], 0.0)


@pytest.mark.parametrize("where", [0, 2100, 4099])
def test_split_update_keeps_the_policy_on_a_nonfinite_cost(where):
    from paper_2104_13542_amd import storm

    prob = _problem(4100, 8, 1.0, 0)
    prob.params.n_null = 0
    eps = inputs.standard_normal(3, (7, 4100, 8))
    eps[2, where, 4] = np.inf
    goal = torch.tensor([1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4, 0.1, 0.45], dtype=torch.float32, device="cuda")
    r = storm.Rollout(prob)
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
        assert after[2] == 1
    finally:
        r.close()


def test_batched_split_update_is_each_problems_own():
    """A batch that mixes both forms of the update: the same bits as plain."""
    from paper_2104_13542_amd import storm

    probs = []
    for k, (n, h) in enumerate([(64, 16), (4100, 8), (513, 64), (1000, 30), (9000, 8), (2049, 1)]):
        pr = inputs.config3_problem(40 + k)
        p = pr.params
        p.n_particles, p.horizon, p.dt, p.n_halton, p.n_null = n, h, np.full(h, 0.02), n // 2, k % 3
        p.beta, p.cov_per_step = [1.0, 50.0, 1e6][k % 3], k % 2
        probs.append(pr)
    goals = torch.tensor([[1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4 + 0.02 * k, 0.1 - 0.03 * k, 0.45]
                          for k in range(len(probs))], dtype=torch.float32, device="cuda")
    b = storm.Batch(probs)
    b.set_config(16, 64, 1)
    plains = [storm.Rollout(pr) for pr in probs]
    try:
        for _ in range(2):
            b.step(goals)
            cmd = b.update(shift=True).clone()
            for k, r in enumerate(plains):
                r.step(goals[k])
                c = r.update(shift=True)[0]
                torch.cuda.synchronize()
                assert torch.equal(cmd[k], c), k
                for x, y in zip(b.get_state(k)[:2], r.get_state()[:2]):
                    np.testing.assert_array_equal(x, y)
    finally:
        b.close()
        for r in plains:
            r.close()
