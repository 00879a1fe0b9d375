"""A captured control step is launched on a raw stream handle (an integer) or,
by default, on the current stream; anything else is refused before the call."""
import ctypes

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture()
def graph():
    from paper_2104_13542_amd import storm

    g = storm.StepGraph.__new__(storm.StepGraph)
    g._h = None  # (a null graph: the call itself ends with STORM_E_NULL)
    g._launch = storm.lib().storm_rollout_graph_launch
    return g


@pytest.mark.parametrize("stream", [b"abc", "abc", 1.5, [1], ctypes.c_void_p(3)])
def test_what_is_no_handle_is_refused(graph, stream):
    with pytest.raises(TypeError):
        graph.launch(stream)


@pytest.mark.parametrize("stream", [0, 7, True])
def test_integers_are_handles(graph, stream):
    from paper_2104_13542_amd import storm

    with pytest.raises(storm.StormError) as e:
        graph.launch(stream)
    assert e.value.code == storm.STORM_E_NULL
