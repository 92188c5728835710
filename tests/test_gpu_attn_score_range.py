"""kvra_chunk_attn on scores far below anything a model makes: every visible score of a row around -1e34, with one key, with
many, split over workgroups and over cut units, in both attention kernels.  All keys before a border are equal, and so are all
keys from it on, with scores half as low: a row that sees none of the latter weighs all its keys alike, every other row weighs
those from the border on alike and the rest not at all.  The products are few-bit numbers times powers of two, so that every
score is exact in fp32 and the expected rows are plain means of V.

Bar: fp32 sums and one rounding to bf16, |err| <= 2^-8 |want| + 1e-4."""
import pytest
import torch

from paper_2405_05329_amd import kvra, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,d,prefix,c,border,tiled", [
    (2, 2, 64, 0, 1, 1, False), (2, 2, 128, 0, 1, 1, False),                                 # a single key
    (8, 2, 128, 449, 63, 480, False), (5, 1, 64, 100, 33, 64, False), (2, 2, 64, 0, 160, 77, False),   # few rows, one workgroup per slice
    (16, 16, 64, 4097, 3, 4098, False), (7, 1, 128, 9000, 4, 5000, False),                   # several
    (71, 1, 64, 700, 900, 1000, True), (32, 32, 128, 0, 2048, 1111, True),                 # many rows, all or most units whole
    (16, 16, 128, 3000, 500, 3200, True), (32, 32, 128, 0, 1024, 640, True), (8, 8, 64, 9000, 1200, 9500, True),   # cut units
])
def test_very_low_scores(H, Hkv, d, prefix, c, border, tiled):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert (kvra.kvra_chunk_attn_row_splits(prefix, c, H, Hkv, d, cus) == 0) == tiled, "not the kernel this shape is here for"
    total = prefix + c
    q = torch.full((c, H, d), -2.0 ** 60, dtype=torch.bfloat16, device="cuda")
    k = torch.full((total, Hkv, d), 2.0 ** 50, dtype=torch.bfloat16, device="cuda")
    k[border:] = 2.0 ** 49
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    v = torch.empty((total, Hkv, d), dtype=torch.bfloat16, device="cuda").normal_(1.0, 1.0, generator=gen)
    out = torch.empty((c, H, d), dtype=torch.bfloat16, device="cuda")
    kvra.kvra_chunk_attn(q, k, v, prefix, c, H, Hkv, d, synth.default_scale(d), out)
    torch.cuda.synchronize()
    below = torch.cat([torch.zeros((1, Hkv, d), dtype=torch.float64, device="cuda"), v.double().cumsum(0)])   # [i]: sum of rows < i
    row = torch.arange(prefix, total, device="cuda")
    first = torch.where(row >= border, border, 0)
    want = (below[row + 1] - below[first]) / (row + 1 - first).double()[:, None, None]
    want = want.repeat_interleave(H // Hkv, dim=1)
    err = (out.double() - want).abs()
    worst = float((err - 2.0 ** -8 * want.abs() - 1e-4).max())
    assert bool(torch.isfinite(out.float()).all()) and worst <= 0, worst
