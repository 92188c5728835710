"""What the calls enqueue, read off a stand-in for the HIP runtime (launch_recorder.py): no GPU."""
import re

import pytest

import test_gpu_layer
import test_gpu_layer_append
import test_gpu_layer_split
import test_gpu_linear_tiles
from paper_2405_05329_amd import kvra
from launch_recorder import layer, linear, record


def _ring(kernel):
    """(tile, rotates, k shared out, starts apart) of a launch of the ring kernel, else None."""
    m = re.match(r"void kvra::linear_kernel<kvra::GemmTile<([^>]*)>, (\w+), (\w+), (\w+)>", kernel)
    return m and (tuple(int(x) for x in m[1].split(",")[:3]), *(x == "true" for x in m.groups()[1:]))


TWO = [(1355, 10912, 1024, "swiglu"), (776, 9984, 2048, "swiglu"), (787, 9824, 8192, "residual"), (982, 8256, 8192, "plain")]


@pytest.mark.parametrize("shape", TWO)
def test_a_linear_call_in_two_launches_enqueues_both_or_none(shape):
    """The second launch's LDS (or the first's) is refused: an error means that nothing was enqueued."""
    assert [(r["rc"], len(r["launches"])) for r in record([linear(*shape)])] == [(kvra.KVRA_OK, 2)]
    for nth in (1, 2):
        assert [(r["rc"], r["launches"]) for r in record([linear(*shape)], refuse_attribute=nth)] == [(kvra.KVRA_ELAUNCH, [])]


def _split(kernel):
    ring = _ring(kernel)
    return ring is not None and ring[2]


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


@pytest.mark.parametrize("m,n,k,mode,apart", [
    # rows a multiple of 4 KB apart, one or three rows within 256 (512 above) of a multiple of 32 KB
    (20, 12288, 8192, "plain", True), (77, 11008, 4096, "swiglu", True), (77, 4096, 11008, "residual", True),
    (40, 4096, 5440, "plain", True), (256, 4096, 16320, "plain", True), (20, 4096, 16384, "plain", True),
    (60, 4096, 8128, "plain", True),
    # rows that lie on many channels: nothing to gain, and up to a fifth to lose
    (20, 12288, 16000, "plain", False), (77, 4096, 16896, "plain", False), (77, 4544, 4544, "residual", False),
    (160, 6144, 5120, "plain", False), (20, 12288, 8064, "plain", False), (77, 4096, 10752, "plain", False),
    # the edges: tokens, depth, weight rows
    (257, 4096, 4096, "plain", False), (20, 4096, 3968, "plain", False), (20, 1024, 8192, "plain", True), (20, 992, 8192, "plain", False),
    (20, 512, 8192, "swiglu", True), (20, 480, 8192, "swiglu", False),
    # forms of the 64 x 64 tiles
    (20, 12288, 12288, "plain", False), (20, 12288, 24576, "plain", True), (160, 6144, 6144, "plain", False), (77, 10240, 6144, "plain", True),
    (182, 8192, 8192, "plain", True),
    # weights beyond the last-level cache and a last token tile that is at most five eighths full
    (144, 12288, 13312, "plain", True), (208, 12288, 13312, "plain", True), (209, 12288, 13312, "plain", False),
    (144, 11264, 11776, "plain", False), (128, 12288, 13312, "plain", False),
])
def test_weight_tiles_start_apart_where_rows_lie_on_few_memory_channels(m, n, k, mode, apart):
    r, = record([linear(m, n, k, mode)])
    assert r["rc"] == kvra.KVRA_OK and [_ring(x["kernel"])[3] for x in r["launches"]] == [apart]


def test_the_gpu_tests_of_tiles_that_start_apart_meet_them():
    shapes = test_gpu_linear_tiles.STARTS_APART
    for shape, r in zip(shapes, record([linear(*s[:4]) for s in shapes])):
        assert [_ring(x["kernel"]) for x in r["launches"]] == [(shape[4][:3], False, False, True)], shape
    shapes = test_gpu_layer_append.STARTS_APART
    for shape, r in zip(shapes, record([layer(hidden, 128, H, Hkv, d, 37, m) for m, H, Hkv, d, hidden, _ in shapes])):
        assert (shape[5], True, False, True) in [_ring(x["kernel"]) for x in r["launches"]], shape


def _waves(launch):
    return launch["block"][0] // 64 if "linear_rows_kernel" in launch["kernel"] else None


@pytest.mark.parametrize("m,n,k,mode,waves", [
    (1, 512, 4096, "plain", 16), (1, 480, 4096, "plain", 8), (1, 1024, 4032, "plain", 8), (16, 512, 11008, "residual", 16),
    (16, 64, 11008, "residual", 8), (4, 256, 4096, "swiglu", 16), (4, 224, 4096, "swiglu", 8), (8, 12288, 4096, "plain", 16),
])
def test_deep_rows_get_sixteen_waves_where_there_are_enough_of_them(m, n, k, mode, waves):
    r, = record([linear(m, n, k, mode)])
    assert r["rc"] == kvra.KVRA_OK and [_waves(x) for x in r["launches"]] == [waves]


def test_the_gpu_tests_of_sixteen_waves_meet_them():
    assert [[_waves(x) for x in r["launches"]] for r in record([linear(*s) for s in test_gpu_linear_tiles.SIXTEEN_WAVES])] == \
        [[16]] * len(test_gpu_linear_tiles.SIXTEEN_WAVES)
    for shape, r in zip(test_gpu_layer_append.SIXTEEN_WAVES,
                        record([layer(hidden, 128, H, Hkv, d, 37, m) for m, H, Hkv, d, hidden in test_gpu_layer_append.SIXTEEN_WAVES])):
        assert _waves(r["launches"][0]) == 16 and "(kvra::RowsKind)2, true" in r["launches"][0]["kernel"], shape


def _normed(launch):
    """(projection, waves, rows and tokens of a block in sixteens) of a launch with the norm inside, else None."""
    m = re.match(r"void kvra::linear_rows_kernel<\(kvra::RowsKind\)(\d), true, (\d+), (\d), (\d)>", launch["kernel"])
    return m and (["plain", "swiglu", "rope"][int(m[1])], int(m[2]), int(m[3]), int(m[4]))


@pytest.mark.parametrize("m,hidden,H,Hkv,d,ffn,qkv,swiglu", [
    # deep rows and few of them, which the norm inside made up to a third slower
    (64, 4096, 1, 1, 64, 256, False, False), (32, 4096, 6, 1, 64, 128, False, False), (128, 3072, 2, 1, 64, 128, False, False),
    (17, 2048, 8, 2, 64, 512, False, False), (48, 1536, 2, 1, 64, 64, False, False), (64, 1280, 2, 1, 64, 64, False, False),
    # the edges of one round of blocks: 1152 columns, 1408 and 1792 from 1024 rows on, 3264 of an odd number of chunks
    (64, 1152, 2, 1, 64, 64, True, True), (64, 1408, 14, 1, 64, 448, True, False), (64, 1792, 14, 1, 64, 512, False, True),
    (64, 1920, 14, 1, 64, 512, False, False), (64, 3264, 2, 1, 64, 64, True, True), (64, 3392, 2, 1, 64, 64, False, False),
    # two rounds up to 832 columns, three up to 128
    (256, 1024, 14, 1, 64, 512, True, True), (257, 1024, 14, 1, 64, 512, False, False), (256, 832, 30, 1, 64, 1024, True, True),
    (257, 832, 30, 1, 64, 1024, False, False), (256, 896, 30, 1, 64, 1024, False, False),
    (384, 128, 30, 1, 64, 1024, True, True), (385, 128, 30, 1, 64, 1024, False, False), (384, 192, 30, 1, 64, 1024, False, False),
    (187, 256, 4, 2, 64, 704, True, True), (160, 1024, 16, 4, 64, 2816, True, False),
])
def test_which_projections_take_the_norm_in_beyond_16_tokens(m, hidden, H, Hkv, d, ffn, qkv, swiglu):
    r, = record([layer(hidden, ffn, H, Hkv, d, 0, m)])
    assert r["rc"] == kvra.KVRA_OK
    inside = {_normed(x)[0] for x in r["launches"] if _normed(x)}
    assert (("rope" in inside), ("swiglu" in inside)) == (qkv, swiglu)


def test_the_gpu_tests_of_the_norm_in_blocks_meet_it():
    shapes = test_gpu_layer_append.NORM_IN_BLOCKS
    met = set()
    for shape, r in zip(shapes, record([layer(hidden, 128, H, Hkv, d, 37, m) for m, H, Hkv, d, hidden in shapes])):
        assert _normed(r["launches"][0])[0] == "rope" and _normed(r["launches"][0])[2:] == (2, 2), shape
        met.add(_normed(r["launches"][0])[1])
    assert met == {8, 16}


def test_the_gpu_tests_of_split_projections_meet_them():
    """Tile, number of shares (off the grid: one workgroup per share and tile, rounded up to eight) and form of the down projection."""
    shapes = test_gpu_layer_split.SPLITS + test_gpu_layer_split.MORE_SPLITS
    results = record([layer(hidden, ffn, H, Hkv, 128, test_gpu_layer_split.PREFIX, m) for m, hidden, ffn, H, Hkv, *_ in shapes])
    for shape, r in zip(shapes, results):
        m, hidden, _, _, _, tile, shares, apart = shape
        down, tiles = r["launches"][-1], -(-hidden // tile[0]) * -(-m // tile[1])
        assert _ring(down["kernel"]) == (tile, False, True, apart), shape
        assert [s for s in range(2, 9) if -(-tiles * s // 8) * 8 == down["grid"][0]] == [shares], shape
    assert {s[6] for s in shapes} == {2, 3, 4, 5, 7, 8}


def test_the_gpu_tests_of_tiles_that_span_three_heads_meet_them():
    shapes = test_gpu_layer_append.THREE_UNITS
    assert {(H + 2 * Hkv) * d % 192 for _, H, Hkv, d, _ in shapes} == {0, 64, 128}
    for shape, r in zip(shapes, record([layer(hidden, 128, H, Hkv, d, 37, m) for m, H, Hkv, d, hidden in shapes])):
        assert ((192, 256, 64), True, False, False) in [_ring(x["kernel"]) for x in r["launches"]], shape


def test_the_gpu_test_of_few_tokens_meets_the_norm_inside():
    met = set()
    for hidden, ffn, H, Hkv, d, _, bounds, swiglu_inside in test_gpu_layer.FEW_TOKENS:
        for r in record([layer(hidden, ffn, H, Hkv, d, lo, hi - lo) for lo, hi in zip(bounds, bounds[1:])]):
            forms = [_normed(x) for x in r["launches"] if _normed(x)]
            assert [f[0] for f in forms] == ["rope"] + ["swiglu"] * swiglu_inside and all(f[2:] == (1, 1) for f in forms), (hidden, ffn)
            met.update(f[:2] for f in forms)
    assert met == {("rope", 8), ("rope", 16), ("swiglu", 8), ("swiglu", 16)}


def test_a_layer_is_five_to_ten_launches():
    """Norms inside the projections, nothing cut in two; and everything apart, with all three of the long projections in two."""
    few, many = record([layer(256, 704, 4, 2, 64, 0, 16), layer(8192, 28672, 64, 64, 128, 0, 1036)])
    assert [len(r["launches"]) for r in (few, many)] == [5, 10]
    assert sum("norm" in x["kernel"] for x in many["launches"]) == 2 and sum(_ring(x["kernel"]) is not None for x in many["launches"]) == 7
