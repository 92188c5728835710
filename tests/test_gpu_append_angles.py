"""The rotation angles of kvra_append_kv: positions up to the largest the library takes, the border between the reduced and
the general form of the angle (2^26, reached with rope bases below 1 only), every tokens-per-workgroup variant with remainders,
with and without queries.  Rotating rows whose low half is 1 and whose high half is 0 gives cos and sin themselves, rounded
to bf16 once: within half a unit in the last place of the exact value (at most 2^-8 of it, plus what one rounding of the fp32 value
before can add)."""
import numpy as np
import pytest
import torch

from paper_2405_05329_amd import kvra
from gpu_pipeline import to_bits
from oracle import kvra_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,prefix,c,base,with_q", [
    (64, 0, 1, 10000.0, True), (128, 0, 5, 10000.0, True), (64, 12345, 3, 10000.0, False), (128, 16000000, 37, 10000.0, True),
    (64, (1 << 24) - 3, 2, 1.0e6, True), (128, 60000, 9, 1.0e-3, True), (64, 1000, 4, 1.0e-9, False),
    (64, 7, 2051, 10000.0, True), (64, 9, 4097, 500000.0, True), (64, 1, 16391, 10000.0, True),
    (128, 3, 2049, 10000.0, True), (128, 0, 8195, 10000.0, True),
])
def test_angles(d, prefix, c, base, with_q):
    H, Hkv, half = 3, 1, d // 2
    one = torch.zeros((c, 1, d), dtype=torch.bfloat16, device="cuda")
    one[..., :half] = 1.0
    kc = torch.zeros((prefix + c, Hkv, d), dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros_like(kc)
    v = torch.randn((c, Hkv, d), device="cuda").bfloat16()
    q = one.expand(c, H, d).contiguous() if with_q else None
    kvra.kvra_append_kv(one, v, q, kc, vc, prefix, c, prefix + c, H, Hkv, d, base)
    torch.cuda.synchronize()
    freq = np.power(float(np.float32(base)), -2.0 * np.arange(half) / d)
    phi = np.arange(prefix, prefix + c, dtype=np.float64)[:, None] * freq
    want = np.concatenate([np.cos(phi), np.sin(phi)], axis=1)
    # pow and the product are rounded differently in other mathematics libraries: two units in the last place of phi
    slack = 2.0 ** -8 * 1.001 * np.abs(want) + 1e-7 + 4 * np.spacing(np.concatenate([phi, phi], axis=1))
    got = orc.bf16_bits_to_f64(to_bits(kc[prefix:]))[:, 0]
    worst = float(np.max(np.abs(got - want) - slack))
    assert worst <= 0, worst
    assert torch.equal(vc[prefix:], v) and not vc[:prefix].any() and not kc[:prefix].any()
    if with_q:
        qb = orc.bf16_bits_to_f64(to_bits(q))
        worst = float(np.max(np.abs(qb - want[:, None]) - slack[:, None]))
        assert worst <= 0, worst


@pytest.mark.parametrize("d,Hkv,prefix,c", [
    (64, 1, 0, 1), (64, 3, 5, 2050), (128, 15, 1, 3), (128, 16, 0, 1), (128, 17, 9, 2), (128, 32, 7, 3),   # 8 .. 512 pieces a token
    (128, 33, 0, 5), (64, 71, 2, 5000), (64, 1, 3, 16500), (128, 49, 0, 4100),
])
def test_copy_without_rotation(d, Hkv, prefix, c):
    """rope_base 0: K and V arrive bit for bit (any pattern, NaNs included), Q and every other row stay as they are."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    bits = lambda *shape: torch.randint(-32768, 32768, shape, dtype=torch.int16, device="cuda", generator=gen)
    k, v, q = bits(c, Hkv, d), bits(c, Hkv, d), bits(c, 2 * Hkv, d)
    kc, vc = bits(prefix + c + 3, Hkv, d), bits(prefix + c + 3, Hkv, d)
    want_k, want_v, want_q = kc.clone(), vc.clone(), q.clone()
    want_k[prefix:prefix + c], want_v[prefix:prefix + c] = k, v
    bf16 = lambda t: t.view(torch.bfloat16)
    kvra.kvra_append_kv(bf16(k), bf16(v), bf16(q), bf16(kc), bf16(vc), prefix, c, prefix + c + 3, 2 * Hkv, Hkv, d, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(kc, want_k) and torch.equal(vc, want_v) and torch.equal(q, want_q)
