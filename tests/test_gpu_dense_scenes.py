"""Scenes of up to 256 obstacles: what the looping and the batched rollout keep of
a scene in LDS leaves room for two workgroups on a compute unit, and cuboids whose
records stay in memory give the same costs (marked gpu)."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs
from tests.gpu_launches import launches, residency

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_13542_amd import storm

    storm.lib()


def _problem(seed, n, h, n_sph, n_box):
    pr = inputs.config3_problem(seed)
    p = pr.params
    p.n_particles, p.horizon, p.dt, p.n_halton, p.n_null = n, h, np.full(h, 0.03), n // 2, 1
    pr.obstacles = inputs.random_scene(np.random.default_rng(seed), n_sph, n_box).astype(np.float32).astype(float)
    return pr


GOAL = [1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4, 0.1, 0.45]
SCENES = [(60, 40), (60, 60), (128, 128), (0, 256), (255, 1)]


@pytest.mark.parametrize("n_sph,n_box", SCENES)
def test_two_workgroups_share_a_compute_unit(n_sph, n_box):
    from paper_2104_13542_amd import storm

    goal = torch.tensor(GOAL, dtype=torch.float32, device="cuda")
    r = storm.Rollout(_problem(1, 300, 64, n_sph, n_box))
    # a dense problem beside a sparse one
    b = storm.Batch([_problem(2, 100, 30, n_sph, n_box), _problem(3, 100, 30, 2, 1)])
    try:
        goals = goal.repeat(2, 1).contiguous()
        for call in (lambda: r.step(goal, C=costs), lambda: b.step(goals)):
            costs = torch.empty(300, device="cuda")
            p, = launches(call)
            assert tuple(p.block) == (512, 1, 1)
            assert residency(p) >= 2
    finally:
        r.close()
        b.close()


# from about 100 cuboids the last ones' records stay in memory
@pytest.mark.parametrize("n_sph,n_box", [(0, 90), (0, 118), (3, 137), (0, 256), (128, 128), (200, 56)])
def test_loop_equals_one_tile_per_workgroup(n_sph, n_box):
    from paper_2104_13542_amd import storm

    goal = torch.tensor(GOAL, dtype=torch.float32, device="cuda")
    r = storm.Rollout(_problem(n_box, 600, 33, n_sph, n_box))
    try:
        for _ in range(2):
            out = r.step(goal, debug=True)
            one, hit = out["C"].clone(), out["terms"][7].clone()
            loop = r.step(goal)["C"].clone()
            r.update(shift=True)
            torch.cuda.synchronize()
            assert torch.any(hit > 0), "the scene should collide somewhere"
            assert torch.equal(one, loop)
    finally:
        r.close()


@pytest.mark.parametrize("n_sph,n_box", [(0, 118), (0, 256), (128, 128)])
def test_batch_of_8_waves_equals_16(n_sph, n_box):
    """The forms add the spheres' penetrations in different orders: 52 terms of
    the cost's own sign, so 52 roundings apart at most on either side."""
    from paper_2104_13542_amd import storm

    b = storm.Batch([_problem(7, 120, 30, n_sph, n_box), _problem(8, 90, 21, 2, 1)])
    goals = torch.tensor([GOAL, GOAL], dtype=torch.float32, device="cuda")
    try:
        got = []
        for waves in (8, 16):
            b.set_config(waves, 64, 1)
            b.step(goals)
            got.append([b.costs(k) for k in range(2)])
        for x, y in zip(*got):
            assert np.all(np.isfinite(x)) and np.max(np.abs(x - y) / np.abs(y)) <= 2 * 52 * 2.0**-24
    finally:
        b.close()
