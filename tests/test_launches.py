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


def _split(kernel):
    return kernel.startswith("void kvra::linear_kernel<") and kernel.split(">")[1].split(",")[2].strip() == "true"


def _attention_uses_scratch(prefix, m, H, Hkv, d, cus=256):
    splits = kvra.kvra_chunk_attn_row_splits(prefix, m, H, Hkv, d, cus)
    return splits > 1 or (splits == 0 and kvra.kvra_chunk_attn_plan(prefix, m, H, Hkv, d, cus)["partial_pieces"] > 0)


# A down projection of 4096 x 11008 wants its k split from 40 to 1000 tokens on
SCRATCH = [(prefix, m, H, Hkv) for prefix, m in ((0, 77), (5824, 77), (2048, 250), (0, 500), (0, 1000), (2048, 1000), (40, 64))
           for H, Hkv in ((32, 32), (32, 8), (32, 1), (8, 8))]


def test_projections_of_a_layer_use_the_scratch_exactly_where_its_attention_does():
    """Calls whose attention leaves the scratch alone may overlap with others; so must their projections."""
    results = record([layer(4096, 11008, H, Hkv, 128, prefix, m) for prefix, m, H, Hkv in SCRATCH])
    met = set()
    for (prefix, m, H, Hkv), r in zip(SCRATCH, results):
        assert r["rc"] == kvra.KVRA_OK
        uses = _attention_uses_scratch(prefix, m, H, Hkv, 128)
        assert any(_split(x["kernel"]) for x in r["launches"]) == uses, (prefix, m, H, Hkv)
        met.add(uses)
    assert met == {True, False}


def test_projections_keep_off_a_scratch_that_the_attention_was_refused():
    """The allocation fails: the attention runs whole units, and what follows does not try again behind its back."""
    assert _attention_uses_scratch(5824, 77, 32, 32, 128)
    r, = record([layer(4096, 11008, 32, 32, 128, 5824, 77)], refuse_malloc=1)
    assert r["rc"] == kvra.KVRA_OK and not any(_split(x["kernel"]) for x in r["launches"])
