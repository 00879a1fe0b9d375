"""Kernel variants that a call selects by its arguments give the same bits:
a step with and without the optional outputs (marked gpu)."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_13542_amd import storm

    storm.lib()


def _goal():
    return torch.tensor([1, 0, 0, 0, -1, 0, 0, 0, -1, 0.4, 0.1, 0.45], dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("make", [lambda: inputs.config1(3), lambda: inputs.config2(3, n_particles=65, horizon=21),
                                  lambda: inputs.config_ball(3, n_particles=33, horizon=9),
                                  lambda: inputs.config_self_mlp(3, n_particles=31, horizon=40)])
def test_step_with_and_without_optional_outputs(make):
    from paper_2104_13542_amd import storm

    got = []
    for debug in (False, True):
        r = storm.Rollout(make())
        try:
            for _ in range(2):
                out = r.step(_goal(), debug=debug)
                cmd, mean, sigma2 = r.update()
            torch.cuda.synchronize()
            got.append([x.cpu().numpy() for x in (out["C"], cmd, mean, sigma2)])
        finally:
            r.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
