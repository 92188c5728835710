"""The tiled attention kernel on launches that it takes (asserted, so that a new dispatch rule cannot empty these tests): its
moving exponent reference, with scores that climb with the key position and scores many times larger than a model's, in whole
units and in cut ones, whose pieces end with references of their own; and odd sizes.  That a reference in force has to move
is worked out from the inputs and asserted too.

Bar of the former: the rounding model's (tests/rounding_model.py) for these very inputs against the fp64 oracle, on rows around
the edges of row tiles and the chunk and some between: every element within six predicted standard deviations, and the mean over
all of them as near to the predicted one as so few rows allow.  (Where a few keys carry a row, their score errors are shared
by all its elements: a row's mean-abs error is then about a half-normal number, whose standard deviation is sqrt(pi/2 - 1)
= 0.756 of its mean e.  The mean over N rows is allowed 4 x 0.756 sqrt(sum e^2) / N more than predicted.)  Of the latter
the parity bar of unit-scale inputs."""
import math

import numpy as np
import pytest
import torch

import rounding_model as rm
from gpu_pipeline import to_bits, to_dev
from oracle import kvra_oracle as orc
from paper_2405_05329_amd import kvra, synth

pytestmark = pytest.mark.gpu

SHAPES = [
    (32, 32, 128, 0, 4096),      # whole units, two rounds
    (32, 8, 128, 700, 2048),     # some units cut
    (16, 4, 128, 2500, 900),     # every unit cut
    (71, 1, 64, 700, 900),       # whole units
    (71, 1, 64, 2000, 500),      # cut
    (16, 16, 64, 3000, 1000),
]


def has_to_move(tops):
    """Whether a row with these largest scores, tile by tile, has its reference moved after the first tile, whose largest it
    is at first: a tile whose weights sum to 2^20 in a lane moves it, and one weight of 2^21 is enough for that."""
    return bool(tops) and max(tops) > tops[0] + 21


def check_launch(H, Hkv, d, prefix, c, q, k, v, scale, label):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert kvra.kvra_chunk_attn_row_splits(prefix, c, H, Hkv, d, cus) == 0, "not the tiled kernel's launch any more"
    out = torch.full((c, H, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    kvra.kvra_chunk_attn(to_dev(q), to_dev(k), to_dev(v), prefix, c, H, Hkv, d, scale, out)
    torch.cuda.synchronize()
    got = orc.bf16_bits_to_f64(to_bits(out))
    assert np.isfinite(got).all()
    plan = kvra.kvra_chunk_attn_plan(prefix, c, H, Hkv, d, cus)
    tile, pieces = plan["key_tile"], kvra.kvra_chunk_attn_pieces(prefix, c, H, Hkv, d, cus)
    rng = np.random.default_rng(5)
    rows = sorted({0, 1, 255, 256, 257, c // 2, c - 33, c - 2, c - 1} | {int(x) for x in rng.integers(0, c, size=50)})
    moved, errors, expected = 0, [], []
    for h in sorted({0, H // 2 - 1, H - 1}):
        g = h // (H // Hkv)
        kf, vf = orc.bf16_bits_to_f64(k[:, g]), orc.bf16_bits_to_f64(v[:, g])
        qf = orc.bf16_bits_to_f64(q[rows, h])
        sig, want = [], []
        for i, r in enumerate(rows):
            t = prefix + r
            s, o = rm.head_sigma(qf[i:i + 1], kf[:t + 1], vf[:t + 1], scale, t, stored_exactly=True)
            sig.append(s[0])
            want.append(o[0])
            score = (kf[:t + 1] @ qf[i]) * scale * math.log2(math.e)
            tops = [score[j:j + tile].max() for j in range(0, t + 1, tile)]
            row_tile = (r * (H // Hkv) + h % (H // Hkv)) // plan["rows_per_tile"]
            moved += any(has_to_move(tops[p["jt0"]:p["jt1"]]) for p in pieces if (p["kv_head"], p["row_tile"]) == (g, row_tile))
        sig, want = np.array(sig), np.array(want)
        err, ulp = np.abs(got[rows, h] - want), rm.bf16_ulp(np.maximum(np.abs(got[rows, h]), np.abs(want)))
        worst = float((err / (rm.K_SIGMA * sig + 0.5 * ulp + 1e-9)).max())
        assert worst <= 1.0, f"{label} head {h}: {worst:.2f} x the elementwise bar"
        errors.append(err.mean(axis=1))
        expected.append(np.sqrt(2.0 / np.pi * (sig * sig + rm.bf16_ulp(want) ** 2 / 12.0)).mean(axis=1))
    assert moved >= 10, f"{label}: the reference of only {moved} of the rows has to move"
    errors, expected = np.concatenate(errors), np.concatenate(expected)
    slack = 4.0 * math.sqrt(math.pi / 2.0 - 1.0) * math.sqrt(float((expected ** 2).sum())) / len(expected)
    print(f"{label}: mean-abs {errors.mean():.3e}, predicted {expected.mean():.3e} + {slack:.3e}")
    assert errors.mean() <= expected.mean() + slack


@pytest.mark.parametrize("step_log2", [0.05, 0.4])
@pytest.mark.parametrize("H,Hkv,d,prefix,c", SHAPES)
def test_rising_scores(H, Hkv, d, prefix, c, step_log2):
    """Scores climb by step_log2 per key, in log2 units: 3 or 26 per 64-key tile."""
    total, rng, scale, qn = prefix + c, np.random.default_rng(9), synth.default_scale(d), 4.0
    u = rng.standard_normal(d).astype(np.float32)
    u /= np.linalg.norm(u)
    ramp = (np.arange(total, dtype=np.float32) * (step_log2 / (scale * math.log2(math.e) * qn)))[:, None, None]
    k = synth.f32_to_bf16_bits(ramp * u + 0.05 * rng.standard_normal((total, Hkv, d), dtype=np.float32))
    q = synth.f32_to_bf16_bits(qn * u + 0.05 * rng.standard_normal((c, H, d), dtype=np.float32))
    v = synth.normal_bf16(9, 61, 2, (total, Hkv, d))
    check_launch(H, Hkv, d, prefix, c, q, k, v, scale, f"rising by {step_log2}")


@pytest.mark.parametrize("H,Hkv,d,prefix,c", SHAPES)
def test_large_scores(H, Hkv, d, prefix, c):
    """Score standard deviation 16 (23 in log2 units): a few keys carry each row."""
    q, k, v = synth.make_qkv(11, 62, prefix + c, H, Hkv, d, q_gain=8.0)
    check_launch(H, Hkv, d, prefix, c, np.ascontiguousarray(q[prefix:]), k, v, 2.0 * synth.default_scale(d), "gain 16")


@pytest.mark.parametrize("H,Hkv,d,prefix,c", [
    (40, 8, 128, 63, 801), (71, 1, 64, 1, 1037),            # whole units, the last row tile a few rows
    (12, 4, 128, 777, 1501), (6, 1, 128, 333, 3001),        # cut units
    (16, 16, 64, 31, 1999), (10, 2, 64, 4095, 1057),
])
def test_ragged_launches(H, Hkv, d, prefix, c):
    """Unit-scale inputs, odd sizes and group sizes, every row.  Rows of the cache behind the valid ones hold NaN, rows around
    the output a value that has to stay, and a second launch has to give the same bits."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert kvra.kvra_chunk_attn_row_splits(prefix, c, H, Hkv, d, cus) == 0, "not the tiled kernel's launch any more"
    total, extra, scale = prefix + c, 140, synth.default_scale(d)
    q, k, v = synth.make_qkv(7, 63, total, H, Hkv, d)
    caches = []
    for rows in (k, v):
        t = torch.full((total + extra, Hkv, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        t[:total] = to_dev(rows)
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
    err = np.abs(got[2:2 + c] - orc.attention_rows(*f64, list(range(prefix, total)), scale))
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
