"""make_robot takes what converts to a number element by element (arrays, lists,
tensors, also those that carry a gradient) and refuses what is too short."""
import numpy as np
import pytest

from paper_2104_13542_amd import inputs

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def storm():
    from paper_2104_13542_amd import storm as s

    return s


DH = np.asarray(inputs.PANDA_DH, dtype=np.float64)
LIMITS = np.linspace(-1.0, -0.4, 7)


class Indexed:
    """A sequence that is indexed by integers only."""

    def __init__(self, values):
        self.values = values

    def __getitem__(self, k):
        return self.values[int(k)]


@pytest.mark.parametrize("name", ["q_min", "q_max", "qd_max"])
@pytest.mark.parametrize("short", [[-1.0], [-1.0] * 6, np.zeros((1, 7)), np.zeros((7, 2)), [None] * 7, 1.0])
def test_limits_that_are_not_seven_numbers_are_refused(storm, name, short):
    with pytest.raises((IndexError, TypeError)):
        storm.make_robot(**{name: short})


@pytest.mark.parametrize("dh", [DH[:1], DH[:7], DH[:, :1], DH[:, :2], DH.reshape(-1), np.zeros((8, 3, 2))])
def test_frames_that_are_not_eight_rows_of_three_are_refused(storm, dh):
    with pytest.raises((IndexError, TypeError)):
        storm.make_robot(dh=dh)


@pytest.mark.parametrize("name", ["q_min", "q_max", "qd_max"])
@pytest.mark.parametrize("given", [list(LIMITS), tuple(LIMITS), LIMITS, LIMITS.reshape(7, 1), torch.tensor(LIMITS),
                                   torch.tensor(LIMITS, requires_grad=True), torch.tensor(LIMITS).bfloat16(),
                                   dict(enumerate(LIMITS)), Indexed(LIMITS), np.concatenate([LIMITS, [9.0, 9.0]])],
                         ids=lambda g: type(g).__name__)
def test_limits_are_taken_element_by_element(storm, name, given):
    r, _ = storm.make_robot(**{name: given})
    want = [np.float32(float(given[j])) for j in range(7)]
    np.testing.assert_array_equal(np.array(getattr(r, name)), want)
    plain, _ = storm.make_robot()
    for other in {"q_min", "q_max", "qd_max"} - {name}:
        np.testing.assert_array_equal(np.array(getattr(r, other)), np.array(getattr(plain, other)))


@pytest.mark.parametrize("dh", [DH + 0.25, (DH + 0.25).tolist(), torch.tensor(DH + 0.25, requires_grad=True),
                                [torch.tensor(row) for row in DH + 0.25], np.concatenate([DH, DH], 1) + 0.25,
                                [list(row) for row in DH[:7] + 0.25] + [list(DH[7] + 0.25) + [1.0]]])
def test_frames_are_taken_element_by_element(storm, dh):
    r, _ = storm.make_robot(dh=dh)
    np.testing.assert_array_equal(np.array(r.dh), (DH + 0.25).astype(np.float32))


def test_default_robot(storm):
    r, _ = storm.make_robot()
    np.testing.assert_array_equal(np.array(r.dh), DH.astype(np.float32))
    for name, want in (("q_min", inputs.PANDA_Q_MIN), ("q_max", inputs.PANDA_Q_MAX), ("qd_max", inputs.PANDA_QD_MAX)):
        np.testing.assert_array_equal(np.array(getattr(r, name)), np.asarray(want, dtype=np.float32))
    assert r.n_spheres == 0 and not r.spheres and not r.self_mlp
