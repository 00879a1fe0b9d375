"""The rollout's looping form (more tiles than compute units) against the
one-tile-per-workgroup form, which the debug outputs take: the same costs bit
for bit, at the tile counts where one gives way to the other, with each option
of the sampling and with scenes on either side of its LDS limit (marked gpu)."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


# 256 tiles are the last that take a workgroup each, 512 the last round of the loop
@pytest.mark.parametrize("n,h,obstacles,comb,cov,null", [
    (256, 64, 20, 0, 0, 0), (257, 64, 20, 0, 0, 2), (333, 37, 25, 1, 1, 2), (512, 33, 100, 0, 1, 0),
    (1026, 30, 3, 1, 0, 1), (1025, 16, 0, 0, 0, 0), (700, 64, 255, 1, 1, 5), (16449, 1, 40, 0, 0, 3)])
def test_loop_equals_one_tile_per_workgroup(n, h, obstacles, comb, cov, null):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_13542_amd import storm

    rng = np.random.default_rng(n)
    pr = inputs.config3_problem(60 + h)
    p = pr.params
    p.n_particles, p.horizon, p.dt, p.n_halton, p.n_null = n, h, np.full(h, 0.03), n // 2, null
    p.comb_filter, p.comb, p.cov_per_step = comb, (0.4, 0.4, 0.2), cov
    pr.obstacles = inputs.random_scene(rng, obstacles // 2, obstacles - obstacles // 2).astype(np.float32).astype(float)
    goal = torch.tensor([1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4, 0.1, 0.45], dtype=torch.float32, device="cuda")
    r = storm.Rollout(pr)
    try:
        for _ in range(2):
            one = r.step(goal, debug=True)["C"].clone()
            loop = r.step(goal)["C"].clone()
            r.update(shift=True)
            torch.cuda.synchronize()
            assert torch.equal(one, loop)
    finally:
        r.close()
