"""What the calls enqueue, read off a stand-in for the HIP runtime (launch_recorder.py): no GPU."""
import pytest

from paper_2405_05329_amd import kvra
from launch_recorder import layer, linear, record


TWO = [(1355, 10912, 1024, "swiglu"), (776, 9984, 2048, "swiglu"), (787, 9824, 8192, "residual"), (982, 8256, 8192, "plain")]


@pytest.mark.parametrize("shape", TWO)
def test_a_linear_call_in_two_launches_enqueues_both_or_none(shape):
    """The second launch's LDS (or the first's) is refused: an error means that nothing was enqueued."""
    assert [(r["rc"], len(r["launches"])) for r in record([linear(*shape)])] == [(kvra.KVRA_OK, 2)]
    for nth in (1, 2):
        assert [(r["rc"], r["launches"]) for r in record([linear(*shape)], refuse_attribute=nth)] == [(kvra.KVRA_ELAUNCH, [])]
