"""The projection that rotates and appends on its way out (inside kvra_layer_chunk): every tile shape of the linear kernel and
the kernel for few tokens (which takes in the norm as well; with 8 and 16 waves), both head sizes, with and without rotation, against the
public operators called one by one.

Bars.  Both sides see the same inputs; they differ where a tensor is rounded to bf16 on one side and not on the other, or
before and after another factor.  rho = 1.66e-3 is the root mean square relative rounding error of bf16.  V: two roundings of
the normed rows (each passed on with relative weight rho) and two of the result, sqrt(4) rho = 3.3e-3, taken as 4e-3; K and Q one
more pair around the rotation, sqrt(6) rho = 4.1e-3, taken as 5e-3; a single element 6 standard deviations of its row's
scale (0.025) and half a unit in the last place of the largest value (0.02): 0.05.  y: the roundings of six stored tensors,
1.2e-2 as for a whole layer.  A swapped pair, row, segment or angle gives 0.1 to 1."""
import pytest
import torch

from paper_2405_05329_amd import kvra, synth

pytestmark = pytest.mark.gpu


def _rel(got, want):
    g, w = got.double(), want.double()
    return float((g - w).norm() / w.norm()), float((g - w).abs().max() / w.square().mean().sqrt())


@pytest.mark.parametrize("m,H,Hkv,d,hidden,tile", [
    (1, 1, 1, 64, 384, (16, 16, 0)), (7, 6, 2, 128, 128, (16, 16, 0)), (16, 71, 1, 64, 192, (16, 16, 0)),
    (1, 3, 1, 64, 4160, (16, 16, 0)), (16, 1, 1, 128, 4096, (16, 16, 0)), (8, 40, 40, 128, 64, (16, 16, 0)),
    # most of these with the norm inside, in blocks of 32 rows and 32 tokens; the tile is what the projection alone would get
    (17, 1, 1, 64, 384, (32, 32, 128)), (17, 1, 1, 128, 128, (32, 32, 128)), (65, 35, 5, 64, 128, (32, 64, 128)),
    (132, 35, 5, 64, 384, (64, 64, 128)), (17, 1, 1, 128, 320, (64, 64, 64)), (31, 4, 2, 64, 2048, (32, 32, 128)),
    (65, 2, 1, 128, 704, (32, 32, 0)), (32, 5, 5, 128, 960, (32, 32, 0)), (20, 1, 1, 64, 4160, (64, 64, 64)),
    # the tiles
    (33, 25, 5, 64, 2176, (32, 32, 128)), (36, 14, 2, 128, 2176, (32, 32, 128)),
    (98, 40, 8, 64, 512, (32, 64, 128)), (33, 40, 8, 128, 512, (32, 64, 128)),
    (388, 15, 5, 64, 256, (64, 64, 64)), (69, 40, 8, 128, 256, (64, 64, 64)),
    (161, 40, 8, 64, 256, (64, 64, 128)), (161, 21, 3, 128, 256, (64, 64, 128)),
    (514, 16, 16, 64, 320, (64, 128, 64)), (193, 40, 8, 128, 320, (64, 128, 64)),
    (782, 24, 8, 64, 384, (128, 128, 64)), (321, 35, 5, 128, 320, (128, 128, 64)),
    (2437, 15, 5, 64, 384, (128, 192, 64)), (642, 35, 5, 128, 384, (128, 192, 64)),
    (3650, 15, 5, 64, 384, (128, 256, 64)), (972, 35, 5, 128, 320, (128, 256, 64)),
    (3106, 24, 8, 64, 384, (192, 192, 64)), (1281, 35, 5, 128, 384, (192, 192, 64)),
    (3666, 15, 5, 128, 384, (192, 256, 64)),
    (2117, 32, 16, 64, 384, (256, 192, 64)), (1154, 40, 8, 128, 384, (256, 192, 64)),
    (3465, 40, 8, 64, 192, (256, 256, 64)), (2700, 25, 5, 128, 384, (256, 256, 64)),
])
@pytest.mark.parametrize("rope_base", [synth.ROPE_BASE, 0.0])
def test_layer_against_its_operators(m, H, Hkv, d, hidden, tile, rope_base):
    rows, ffn, prefix, scale = (H + 2 * Hkv) * d, 128, 37, synth.default_scale(d)
    assert kvra.kvra_linear_tile(m, rows, hidden, False)[:3] == tile
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)

    def normal(*shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(mean, std, generator=gen)

    x, n1, n2 = normal(m, hidden), normal(hidden, std=0.1, mean=1.0), normal(hidden, std=0.1, mean=1.0)
    wqkv, wo = normal(rows, hidden, std=hidden ** -0.5), normal(hidden, H * d, std=(H * d) ** -0.5)
    wg, wu, wd = normal(ffn, hidden, std=hidden ** -0.5), normal(ffn, hidden, std=hidden ** -0.5), normal(hidden, ffn, std=ffn ** -0.5)
    layer = kvra.make_layer(hidden, ffn, H, Hkv, d, synth.RMS_EPS, rope_base, scale, n1, wqkv, wo, n2, wg, wu, wd)
    cap = prefix + m + 3
    kc, vc = normal(cap, Hkv, d), normal(cap, Hkv, d)
    kc2, vc2 = kc.clone(), vc.clone()
    before_k, before_v = kc.clone(), vc.clone()
    y = torch.full((m, hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
    nbytes = kvra.kvra_layer_workspace_bytes(layer, m)
    ws = torch.full((nbytes + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    kvra.kvra_layer_chunk(layer, x, y, kc, vc, prefix, m, cap, ws, nbytes)
    torch.cuda.synchronize()
    assert bool((ws[nbytes:] == 0xFF).all()), "wrote behind the workspace"

    h, q = torch.empty_like(x), torch.empty((m, H, d), dtype=torch.bfloat16, device="cuda")
    k, v, out = torch.empty((m, Hkv, d), dtype=torch.bfloat16, device="cuda"), normal(m, Hkv, d), torch.empty_like(q)
    x2, act, want = torch.empty_like(x), normal(m, ffn), torch.empty_like(x)
    kvra.kvra_rms_norm(x, n1, h, m, hidden, synth.RMS_EPS)
    kvra.kvra_qkv_proj(h, wqkv, q, k, v, m, H, Hkv, d, hidden)
    kvra.kvra_append_kv(k, v, q, kc2, vc2, prefix, m, cap, H, Hkv, d, rope_base)
    kvra.kvra_chunk_attn(q, kc2, vc2, prefix, m, H, Hkv, d, scale, out)
    kvra.kvra_linear(out, wo, None, x, x2, m, hidden, H * d)
    kvra.kvra_rms_norm(x2, n2, h, m, hidden, synth.RMS_EPS)
    kvra.kvra_linear(h, wg, wu, None, act, m, ffn, hidden)
    kvra.kvra_linear(act, wd, None, x2, want, m, hidden, ffn)
    torch.cuda.synchronize()

    for got, ref, old, bar, label in ((kc, kc2, before_k, 5e-3, "K"), (vc, vc2, before_v, 4e-3, "V")):
        assert torch.equal(got[:prefix], old[:prefix]) and torch.equal(got[prefix + m:], old[prefix + m:]), label
        rel, worst = _rel(got[prefix:prefix + m], ref[prefix:prefix + m])
        assert rel <= bar and worst <= 0.05, f"{label}: {rel:.2e}, worst element {worst:.3f}"
    rel, worst = _rel(y, want)
    assert rel <= 1.2e-2, f"y: {rel:.2e}"


# weight tiles that start along k apart: every tile up to 256 tokens, with stages of 64 and 128 and odd numbers of them
STARTS_APART = [
    (20, 30, 5, 64, 4096, (32, 32, 128)), (33, 6, 1, 128, 5504, (32, 32, 128)), (33, 60, 15, 64, 5504, (32, 64, 128)),
    (33, 25, 5, 128, 4096, (32, 64, 128)), (33, 14, 1, 64, 5440, (64, 64, 64)), (33, 6, 1, 128, 5440, (64, 64, 64)),
    (193, 25, 5, 64, 4096, (64, 64, 128)), (20, 32, 32, 128, 5504, (64, 64, 128)), (193, 60, 15, 64, 5504, (64, 128, 64)),
    (77, 32, 32, 128, 4096, (64, 128, 64)), (129, 140, 28, 64, 5504, (128, 128, 64)), (129, 32, 32, 128, 4096, (128, 128, 64)),
]


@pytest.mark.parametrize("m,H,Hkv,d,hidden,tile", STARTS_APART)
def test_layer_whose_projection_starts_its_tiles_apart(m, H, Hkv, d, hidden, tile):
    """(That these calls get that form is asserted in tests/test_launches.py, by the same list.)"""
    test_layer_against_its_operators(m, H, Hkv, d, hidden, tile, synth.ROPE_BASE)


# few tokens on deep rows and enough of them: the norm inside, 16 waves (below 1024 rows, as above, 8)
SIXTEEN_WAVES = [(1, 14, 1, 64, 4160), (16, 6, 1, 128, 4096), (5, 20, 5, 64, 5504)]


@pytest.mark.parametrize("m,H,Hkv,d,hidden", SIXTEEN_WAVES)
@pytest.mark.parametrize("rope_base", [synth.ROPE_BASE, 0.0])
def test_layer_whose_projection_takes_sixteen_waves(m, H, Hkv, d, hidden, rope_base):
    test_layer_against_its_operators(m, H, Hkv, d, hidden, (16, 16, 0), rope_base)


# the norm inside, in blocks of 32 rows and 32 tokens, at the edges of its rule: one round of blocks to three, the deepest rows (of which
# the waves keep two chunks each and read the others again), 8 waves and 16
NORM_IN_BLOCKS = [
    (17, 1, 1, 64, 64), (127, 30, 1, 64, 1024), (33, 60, 2, 64, 1152), (31, 4, 2, 64, 1088), (100, 14, 1, 128, 2112), (17, 3, 3, 128, 3264),
    (125, 60, 2, 64, 832), (113, 26, 1, 128, 448), (32, 14, 1, 64, 1408), (132, 24, 6, 128, 128),
]


@pytest.mark.parametrize("m,H,Hkv,d,hidden", NORM_IN_BLOCKS)
def test_layer_with_the_norm_in_blocks(m, H, Hkv, d, hidden):
    """(That these calls get that form is asserted in tests/test_launches.py, by the same list.)"""
    tile = kvra.kvra_linear_tile(m, (H + 2 * Hkv) * d, hidden, False)[:3]
    test_layer_against_its_operators(m, H, Hkv, d, hidden, tile, synth.ROPE_BASE)


# 96 weight rows to a wave, three units of 32: with head_dim 64 a tile spans three heads, and the two waves' third units are the halves
# of the middle one; rows that fill the last tile, and that leave it a third and two thirds full
THREE_UNITS = [(1925, 64, 16, 64, 256), (3651, 35, 7, 64, 256), (1737, 99, 1, 64, 320)]


@pytest.mark.parametrize("m,H,Hkv,d,hidden", THREE_UNITS)
@pytest.mark.parametrize("rope_base", [synth.ROPE_BASE, 0.0])
def test_layer_whose_tiles_span_three_heads(m, H, Hkv, d, hidden, rope_base):
    test_layer_against_its_operators(m, H, Hkv, d, hidden, (192, 256, 64), rope_base)
