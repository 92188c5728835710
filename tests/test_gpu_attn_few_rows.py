"""kvra_chunk_attn on launches of few rows, where the kernel whose waves share out the keys takes over: edges of its slices
(32 rows) and key tiles (64 keys), fewer tiles than waves, one and several workgroups per slice up to the largest count,
(head, split) pairs dealt over the XCDs or not, whole and partial rounds of workgroups, both head sizes.

Bar: the parity bar of unit-scale inputs against the fp64 oracle.  Rows of the cache behind the valid ones hold NaN, rows
around the output a value that has to stay, and a second launch has to give the same bits."""
import numpy as np
import pytest
import torch

from oracle import kvra_oracle as orc
from paper_2405_05329_amd import kvra, synth
from gpu_pipeline import to_bits, to_dev

pytestmark = pytest.mark.gpu


BEYOND = [(16, 16, 128, 12000, 130), (8, 8, 64, 20000, 420), (8, 8, 128, 20000, 290)]   # tiles with waves that have no rows


@pytest.mark.parametrize("H,Hkv,d,prefix,c", [
    (2, 2, 64, 0, 1), (2, 2, 64, 63, 1), (3, 3, 128, 0, 31), (3, 3, 128, 31, 33), (5, 1, 128, 64, 32),   # one tile, two tiles
    (8, 8, 64, 447, 65), (8, 8, 128, 448, 64), (8, 2, 128, 449, 63),          # eight tiles, and one more or less
    (16, 4, 64, 511, 129), (71, 1, 64, 300, 30),                              # whole rounds and a partial one, odd groups
    (8, 2, 128, 1699, 300), (8, 2, 128, 777, 524), (4, 2, 64, 2500, 179),     # two and three workgroups per slice
    (32, 32, 128, 5824, 77), (32, 32, 128, 8000, 1), (16, 16, 64, 4097, 3),   # eight heads or more: pairs by XCD
    (7, 1, 64, 23000, 2), (8, 1, 128, 19999, 4),                              # the most workgroups per slice
    *BEYOND,                                                                  # the first ones that go to the tiled kernel
])
def test_few_rows(H, Hkv, d, prefix, c):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiled = kvra.kvra_chunk_attn_row_splits(prefix, c, H, Hkv, d, cus) == 0
    assert tiled == ((H, Hkv, d, prefix, c) in BEYOND), "not the kernel this shape is here for"
    C, extra = prefix + c, 40
    q, k, v = synth.make_qkv(6, 51, C, H, Hkv, d)
    scale = synth.default_scale(d)
    caches = []
    for rows in (k, v):
        t = torch.full((C + extra, Hkv, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        t[:C] = to_dev(rows)
        caches.append(t)
    outs = []
    for _ in range(2):
        buf = torch.full((c + 4, H, d), 7.0, dtype=torch.bfloat16, device="cuda")
        kvra.kvra_chunk_attn(to_dev(q[prefix:]), *caches, prefix, c, H, Hkv, d, scale, buf[2:2 + c])
        torch.cuda.synchronize()
        outs.append(to_bits(buf))
    assert np.array_equal(outs[0], outs[1])
    got = orc.bf16_bits_to_f64(outs[0])
    assert np.all(got[:2] == 7.0) and np.all(got[2 + c:] == 7.0), "wrote outside the output"
    f64 = [orc.bf16_bits_to_f64(t) for t in (q, k, v)]
    err = np.abs(got[2:2 + c] - orc.attention_rows(*f64, list(range(prefix, C)), scale))
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
