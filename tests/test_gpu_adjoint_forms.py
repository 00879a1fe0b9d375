"""The adjoint's forms (a tile per workgroup, a tile per wavefront, two runs per
wavefront) at the tile counts where one gives way to the next: the gradient
against the FP64 oracle, and the batched refinement, whose launches mix the
forms, against each problem's own (marked gpu)."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs
from tests.test_gpu_adjoint import _dev, _setup
from tests.gpu_common import f32

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_13542_amd import storm

    storm.lib()


# 512 tiles are the last that are split over a workgroup each, 2048 the last
# that take four runs per chunk; H = 64, 33: one particle and no or many idle lanes
@pytest.mark.parametrize("N,H,n_null", [(1024, 30, 0), (1026, 30, 1), (513, 33, 3), (2048, 64, 0), (2049, 64, 2),
                                        (8200, 15, 0), (16400, 8, 5), (70000, 1, 0)])
def test_gradient_at_the_forms_edges(oracle_lib, N, H, n_null):
    from paper_2104_13542_amd import storm

    mask = inputs.COST_POSE | inputs.COST_JOINT | inputs.COST_VEL | inputs.COST_STOP
    prob, o, eps, mean = _setup(oracle_lib, N=N, H=H, mask=mask, n_null=n_null)
    r = storm.Rollout(prob)
    try:
        g, J = r.grad(_dev(mean), _dev(o.goal), noise=_dev(eps.transpose(2, 0, 1)))
        torch.cuda.synchronize()
        gg, J = g.cpu().double().numpy(), J.item()
    finally:
        r.close()
    eps_o = eps.copy()
    eps_o[N - n_null:] = 0.0
    g_ref, J_ref = o.grad(mean, np.sqrt(f32(np.asarray(prob.params.sigma_init) ** 2)), eps_o)
    # the tolerances of the adjoint's other gradient tests
    assert abs(J - J_ref) <= 1e-4 * abs(J_ref)
    assert np.linalg.norm(gg - g_ref) <= 1e-3 * np.linalg.norm(g_ref)
    assert np.max(np.abs(gg - g_ref)) <= 1e-3 * np.max(np.abs(g_ref))


@pytest.mark.parametrize("shapes", [[(500, 30), (3, 64), (333, 37), (64, 16), (1, 1), (511, 33)],
                                    [(1024, 30), (1026, 30), (40, 7), (16400, 8)]])
def test_batched_refinement_is_each_problems_own(shapes):
    from paper_2104_13542_amd import storm

    probs = []
    for k, (n, h) in enumerate(shapes):
        pr = inputs.config3_problem(20 + k)
        p = pr.params
        p.n_particles, p.horizon, p.dt, p.n_halton, p.n_null = n, h, np.full(h, 0.02), n // 2, min(k % 3, n - 1)
        p.grad_mask = inputs.COST_POSE | inputs.COST_JOINT | (inputs.COST_VEL if k % 2 else 0)
        probs.append(pr)
    goals = torch.tensor([[1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4 + 0.02 * k, 0.1 - 0.03 * k, 0.45]
                          for k in range(len(probs))], dtype=torch.float32, device="cuda")
    b = storm.Batch(probs)
    b.set_config(16, 64, 1)
    plains = [storm.Rollout(pr) for pr in probs]
    try:
        b.step(goals)
        cmd = b.refine(goals, iterations=3, lr=0.05, shift=True).clone()
        for k, r in enumerate(plains):
            r.step(goals[k])
            c = r.refine(goals[k], iterations=3, lr=0.05, shift=True).clone()
            torch.cuda.synchronize()
            assert torch.equal(cmd[k], c), shapes[k]
            np.testing.assert_array_equal(b.get_state(k)[0], r.get_state()[0])
    finally:
        b.close()
        for r in plains:
            r.close()
