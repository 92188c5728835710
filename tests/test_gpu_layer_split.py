"""Down projections whose k is shared out over workgroups (inside kvra_layer_chunk, where the attention of the call uses the
scratch): 64 x 128, 128 x 128 and 128 x 256 tiles with two to eight shares (even and odd numbers, and more than the merge adds in one
go), ragged tokens, and k stages that do not divide evenly.  That the calls are split so is asserted in tests/test_launches.py, by the
same lists; here, that the device is the one those numbers are for.

Against the public operators one by one, which never split: y differs by roundings of stored tensors (1.2e-2 relative, as for
a whole layer; a lost or doubled share is of order 1).  The pieces of a tile may finish in any order; the sums are taken in
the order of the shares, so repeated calls, which also find the counters as the call before left them, agree bit for bit."""
import pytest
import torch

from paper_2405_05329_amd import kvra, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,ffn,H", [(77, 11008, 8), (250, 11008, 8), (333, 11072, 8), (500, 8256, 8), (1000, 11008, 32)])
def test_layer_with_a_split_down_projection(m, ffn, H):
    check_split(m, 4096, ffn, H, H)


PREFIX = 2048
# tokens, hidden, ffn, heads, tile, shares, whether the weight tiles start apart
SPLITS = [
    (77, 4096, 11008, 8, 8, (64, 128, 64), 4, True), (250, 4096, 11008, 8, 8, (128, 128, 64), 4, True),
    (333, 4096, 11072, 8, 8, (128, 128, 64), 2, False), (500, 4096, 8256, 8, 8, (128, 128, 64), 2, False),
    (1000, 4096, 11008, 32, 32, (128, 256, 64), 2, False),
]
MORE_SPLITS = [
    (77, 1024, 11008, 8, 8, (64, 128, 64), 8, True), (40, 2048, 8256, 8, 8, (64, 128, 64), 7, True),
    (100, 3072, 8192, 8, 8, (64, 128, 64), 5, True), (77, 5120, 13824, 8, 8, (64, 128, 64), 3, False),
    (333, 1024, 8192, 8, 2, (64, 128, 64), 5, False), (300, 2048, 8256, 8, 8, (128, 128, 64), 5, False),
    (333, 3072, 8192, 8, 8, (128, 128, 64), 3, False), (1200, 2048, 11008, 16, 16, (128, 256, 64), 3, False),
]


@pytest.mark.parametrize("m,hidden,ffn,H,Hkv,tile,shares,apart", MORE_SPLITS)
def test_layer_with_other_numbers_of_shares(m, hidden, ffn, H, Hkv, tile, shares, apart):
    check_split(m, hidden, ffn, H, Hkv)


def check_split(m, hidden, ffn, H, Hkv):
    d, prefix, scale = 128, PREFIX, synth.default_scale(128)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m)

    def normal(*shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(mean, std, generator=gen)

    rows = (H + 2 * Hkv) * d
    x, n1, n2 = normal(m, hidden), normal(hidden, std=0.1, mean=1.0), normal(hidden, std=0.1, mean=1.0)
    wqkv, wo = normal(rows, hidden, std=hidden ** -0.5), normal(hidden, H * d, std=(H * d) ** -0.5)
    wg, wu, wd = normal(ffn, hidden, std=hidden ** -0.5), normal(ffn, hidden, std=hidden ** -0.5), normal(hidden, ffn, std=ffn ** -0.5)
    layer = kvra.make_layer(hidden, ffn, H, Hkv, d, synth.RMS_EPS, synth.ROPE_BASE, scale, n1, wqkv, wo, n2, wg, wu, wd)
    kc, vc = normal(prefix + m, Hkv, d), normal(prefix + m, Hkv, d)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus == 256
    assert kvra.kvra_chunk_attn_plan(prefix, m, H, Hkv, d, cus)["partial_pieces"] > 0
    assert kvra.kvra_chunk_attn_row_splits(prefix, m, H, Hkv, d, cus) != 1   # the attention uses the scratch
    nbytes = kvra.kvra_layer_workspace_bytes(layer, m)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    ys = []
    for _ in range(4):
        y = torch.full((m, hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
        kvra.kvra_layer_chunk(layer, x, y, kc, vc, prefix, m, prefix + m, ws, nbytes)
        ys.append(y)
    torch.cuda.synchronize()
    assert all(torch.equal(ys[0], y) for y in ys[1:])

    h, q = torch.empty_like(x), torch.empty((m, H, d), dtype=torch.bfloat16, device="cuda")
    k, v, out = torch.empty((m, Hkv, d), dtype=torch.bfloat16, device="cuda"), normal(m, Hkv, d), torch.empty_like(q)
    x2, act, want = torch.empty_like(x), normal(m, ffn), torch.empty_like(x)
    kvra.kvra_rms_norm(x, n1, h, m, hidden, synth.RMS_EPS)
    kvra.kvra_qkv_proj(h, wqkv, q, k, v, m, H, Hkv, d, hidden)
    kvra.kvra_append_kv(k, v, q, kc, vc, prefix, m, prefix + m, H, Hkv, d, synth.ROPE_BASE)
    kvra.kvra_chunk_attn(q, kc, vc, prefix, m, H, Hkv, d, scale, out)
    kvra.kvra_linear(out, wo, None, x, x2, m, hidden, H * d)
    kvra.kvra_rms_norm(x2, n2, h, m, hidden, synth.RMS_EPS)
    kvra.kvra_linear(h, wg, wu, None, act, m, ffn, hidden)
    kvra.kvra_linear(act, wd, None, x2, want, m, hidden, ffn)
    torch.cuda.synchronize()
    rel = float((ys[0].double() - want.double()).norm() / want.double().norm())
    assert rel <= 1.2e-2, f"y: {rel:.2e}"
