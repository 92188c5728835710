"""kvra_linear over the range of its launch rule: every tile shape of the ring kernel (sizes at which the rule picks it,
ragged in tokens and columns), one k stage only, several tiles per workgroup, odd numbers of stages, and the direct
kernel for few tokens at the edges of its range.  (That the rule picks them is asserted: here, and for the first list in
tests/test_library_host.py.)

Bar as for every single operator: fp32 arithmetic and one rounding to bf16, |err| <= 2^-8 |want| + 1e-4 against the
fp64 oracle (half a unit in the last place is at most 2^-8 of the value; the fp32 sums over k <= 5632 unit-variance terms
are good to 1e-5)."""
import numpy as np
import pytest
import torch

from oracle import kvra_oracle as orc
from paper_2405_05329_amd import kvra, synth
from gpu_pipeline import to_bits, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,mode", [
    (2221, 5408, 192, "residual"), (1435, 4128, 192, "swiglu"),      # 256 x 256
    (4093, 2144, 192, "plain"), (849, 4960, 192, "swiglu"),          # 256 x 192
    (2691, 4384, 192, "residual"),                                   # 192 x 256
    (2317, 3360, 192, "residual"), (649, 5472, 192, "swiglu"),       # 192 x 192
    (3789, 1568, 320, "plain"), (389, 5472, 384, "swiglu"),          # 128 x 256
    (813, 4768, 192, "residual"), (527, 3424, 192, "swiglu"),        # 128 x 192
    (321, 5728, 192, "plain"), (195, 4384, 192, "swiglu"),           # 128 x 128
    (325, 4896, 192, "residual"), (197, 3680, 192, "swiglu"),        # 64 x 128
    (77, 96, 192, "residual"), (77, 96, 192, "swiglu"),              # 64 x 64, k stages of 64
    (77, 4576, 384, "plain"), (131, 1376, 384, "swiglu"),            # 64 x 64, k shared out over two waves
    (97, 2080, 384, "residual"), (77, 1440, 384, "swiglu"),          # 32 x 64
    (39, 96, 384, "residual"), (39, 32, 384, "swiglu"),              # 32 x 32
    (5000, 4096, 64, "residual"), (4001, 2080, 64, "swiglu"),        # 128 x 128, one stage per tile, several tiles per workgroup
    (6001, 4128, 128, "plain"),                                      # 128 x 128, several tiles of two stages
    (1, 32, 64, "plain"), (16, 544, 320, "residual"), (8, 8224, 128, "plain"), (9, 8224, 128, "residual"),
    (5, 1056, 5632, "residual"), (17, 544, 320, "plain"), (1, 64, 128, "swiglu"),   # few tokens
    (17, 96, 128, "swiglu"), (16, 2080, 320, "swiglu"), (16, 4064, 64, "swiglu"), (8, 4128, 576, "swiglu"),   # SwiGLU: direct
    (9, 4128, 64, "swiglu"), (4, 8224, 576, "swiglu"), (5, 8224, 64, "swiglu"), (3, 32, 4608, "swiglu"),      # or tiled
])
def test_linear_tiles(m, n, k, mode):
    check_linear(m, n, k, mode)


@pytest.mark.parametrize("m,n,k,mode,tile", [
    (3746, 8768, 64, "plain", (256, 192, 64, 3)), (2564, 6272, 64, "swiglu", (256, 192, 64, 3)),
    (2761, 8768, 64, "swiglu", (256, 256, 64, 3)), (5716, 5024, 128, "plain", (256, 256, 64, 2)),
    (3549, 6688, 128, "residual", (192, 256, 64, 2)), (2564, 6272, 320, "plain", (192, 192, 64, 2)),
    (5519, 2944, 320, "residual", (128, 256, 64, 2)), (4140, 2944, 384, "plain", (128, 192, 64, 2)),
])
def test_tiles_in_turn(m, n, k, mode, tile):
    """The interleaved form of the ring kernel (the six larger tiles) with several tiles per workgroup: the loads run on into
    the next tile while the last one is finished, with one stage per tile, two, and numbers at which the ring does not come
    out even."""
    assert kvra.kvra_linear_tile(m, n, k, mode == "swiglu") == tile
    check_linear(m, n, k, mode)


@pytest.mark.parametrize("m,n,k,mode,tile", [
    (26, 32, 4224, "plain", (32, 32, 128, 1)), (35, 32, 4288, "swiglu", (64, 64, 64, 1)), (33, 4192, 4224, "residual", (32, 64, 128, 1)),
    (129, 10400, 4096, "plain", (64, 64, 128, 2)), (67, 8224, 4224, "swiglu", (128, 128, 64, 1)),
    (129, 8608, 4096, "swiglu", (128, 192, 64, 1)),
])
def test_weight_tiles_that_start_apart(m, n, k, mode, tile):
    """Up to 256 tokens on rows of 4096 and more: the range in which weight tiles may start their walk along k apart (those of 4096
    do, the others' rows lie on many memory channels)."""
    assert kvra.kvra_linear_tile(m, n, k, mode == "swiglu") == tile
    check_linear(m, n, k, mode)


STARTS_APART = [
    (26, 1024, 5504, "plain", (32, 32, 128, 1)), (35, 1024, 5440, "swiglu", (64, 64, 64, 1)), (33, 4192, 5504, "residual", (32, 64, 128, 1)),
    (67, 8224, 5504, "swiglu", (128, 128, 64, 1)), (100, 12288, 5504, "plain", (64, 128, 64, 1)),
    (200, 11008, 4096, "swiglu", (128, 256, 64, 1)), (256, 1056, 16320, "residual", (64, 64, 64, 1)),
]


@pytest.mark.parametrize("m,n,k,mode,tile", STARTS_APART)
def test_weight_tiles_that_do_start_apart(m, n, k, mode, tile):
    """Every weight tile starts its walk along k elsewhere and wraps around: stages of 64 and 128, an odd number of them.  (That
    these calls get that form is asserted in tests/test_launches.py, by the same list.)"""
    assert kvra.kvra_linear_tile(m, n, k, mode == "swiglu") == tile
    check_linear(m, n, k, mode)


@pytest.mark.parametrize("m,n,k,mode,tile", [
    (1355, 10912, 1024, "swiglu", (256, 256, 64, 2)), (776, 9984, 2048, "swiglu", (192, 192, 64, 2)),
    (787, 9824, 8192, "residual", (192, 192, 64, 1)), (982, 8256, 8192, "plain", (128, 256, 64, 1)),
])
def test_launches_in_two(m, n, k, mode, tile):
    """Calls whose tiles would leave their last round nearly empty: whole rounds of one tile, then another on the columns left."""
    got = kvra.kvra_linear_tile(m, n, k, mode == "swiglu")
    assert got == tile and -(-n * (2 if mode == "swiglu" else 1) // got[0]) * -(-m // got[1]) > 256 * got[3]   # not all of it
    check_linear(m, n, k, mode)


@pytest.mark.parametrize("m,n,k", [(17, 32, 448), (63, 96, 576), (400, 256, 704), (1000, 256, 704), (33, 4096, 960), (300, 800, 832)])
@pytest.mark.parametrize("mode", ["plain", "residual"])
def test_blocks_of_32_tokens(m, n, k, mode):
    """The direct kernel beyond 16 tokens, where k is an odd number of 64-column chunks (8 and 16 waves, up to one round)."""
    assert kvra.kvra_linear_tile(m, n, k, False) == (32, 32, 0, 1)
    check_linear(m, n, k, mode)


def check_linear(m, n, k, mode):
    x = synth.normal_bf16(5, 23, 0, (m, k))
    w = synth.normal_bf16(5, 23, 1, (n, k), std=k ** -0.5)
    xf, wf = orc.bf16_bits_to_f64(x), orc.bf16_bits_to_f64(w)
    want = orc.linear(xf, wf)
    w2 = res = None
    if mode == "residual":
        r = synth.normal_bf16(5, 23, 2, (m, n))
        res = to_dev(r)
        want = want + orc.bf16_bits_to_f64(r)
    elif mode == "swiglu":
        u = synth.normal_bf16(5, 23, 3, (n, k), std=k ** -0.5)
        w2 = to_dev(u)
        want = orc.silu(want) * orc.linear(xf, orc.bf16_bits_to_f64(u))
    pad = 64                                           # rows before and after the output that no launch may touch
    buf = torch.full((m + 2 * pad, n), 7.0, dtype=torch.bfloat16, device="cuda")
    kvra.kvra_linear(to_dev(x), to_dev(w), w2, res, buf[pad:pad + m], m, n, k)
    torch.cuda.synchronize()
    got = orc.bf16_bits_to_f64(to_bits(buf))
    assert np.all(got[:pad] == 7.0) and np.all(got[pad + m:] == 7.0), "wrote outside the output"
    err = np.abs(got[pad:pad + m] - want)
    worst = np.max(err - (2.0 ** -8 * np.abs(want) + 1e-4))
    assert worst <= 0, f"{mode} {m}x{n}x{k}: exceeds the one-rounding bound by {worst:.3e} (max err {err.max():.3e})"


SIXTEEN_WAVES = [(1, 1024, 4096, "plain"), (16, 1056, 5632, "residual"), (3, 544, 4608, "swiglu"), (8, 12288, 4160, "plain")]


@pytest.mark.parametrize("m,n,k,mode", SIXTEEN_WAVES)
def test_few_tokens_on_many_deep_rows(m, n, k, mode):
    """The direct kernel with 16 waves: chunks that come out even over them and ones that do not."""
    check_linear(m, n, k, mode)
