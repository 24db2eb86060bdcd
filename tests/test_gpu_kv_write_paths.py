"""KV cache writes over both thread mappings and the quotient's whole range: every finite bf16 value against scales
on both sides of where the corrected reciprocal takes over from the division.  Codes are bit for bit."""
import numpy as np
import pytest
import torch

from oracle import kv
from tests.gpu_util import announce, assert_codes_equal, need_gpu, u16, u8

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp8rl():
    need_gpu()
    import paper_2601_18150_amd as m
    m.load()
    return m


def write(fp8rl, k, v, slots, nb, ks, vs):
    kvh = k.shape[1]
    kc = torch.full((nb, kvh, 16, 128), 0x55, dtype=torch.uint8, device="cuda")
    vc = torch.full((nb, kvh, 4, 128, 4), 0x55, dtype=torch.uint8, device="cuda")
    one = lambda s: torch.tensor([s], dtype=torch.float32, device="cuda")
    fp8rl.fp8rl_kv_cache_write_fp8(k.cuda(), v.cuda(), torch.from_numpy(slots).cuda(), one(ks), one(vs), kc, vc)
    torch.cuda.synchronize()
    kr, vr = np.full(kc.shape, 0x55, np.uint8), np.full(vc.shape, 0x55, np.uint8)
    real = slots >= 0                             # (negative slots are padding)
    kv.write_cache(kr, vr, u16(k)[real], u16(v)[real], slots[real], np.float32(ks), np.float32(vs))
    assert_codes_equal(u8(kc), kr, f"k codes, scale {ks!r}")
    assert_codes_equal(u8(vc), vr, f"v codes, scale {vs!r}")


@pytest.mark.parametrize("copies", [1, 17])       # 510 (token, head) pairs: one token per thread; 8670: four
@pytest.mark.parametrize("scales", [(0.0123, 3.7e-4), (2.0 ** -91, float(np.nextafter(np.float32(2.0 ** -91), np.float32(0)))),
                                    (2.0 ** 110, float(np.nextafter(np.float32(2.0 ** 110), np.float32(1e38)))),
                                    (1.0, 0.33333334), (1e-40, 3e38), (7.0e-5, 1.7e3)])
def test_every_value_and_scale_range(fp8rl, scales, copies):
    announce(f"kv write every bf16 value, scales {scales}, {copies} heads")
    bits = np.array([b for b in range(1 << 16) if (b & 0x7F80) != 0x7F80], np.uint16)
    x = torch.from_numpy(bits.view(np.int16).copy()).view(torch.bfloat16).reshape(-1, 1, 128).repeat(1, copies, 1).contiguous()
    t = x.shape[0]
    with np.errstate(over="ignore"):
        write(fp8rl, x, x.flip(0).contiguous(), np.arange(t, dtype=np.int64), (t + 15) // 16, *scales)


@pytest.mark.parametrize("tokens,kv_heads", [(1, 1), (4, 1024), (5, 1024), (1023, 8), (1024, 8), (1025, 8), (1027, 8), (2050, 4)])
def test_both_mappings_at_their_border(fp8rl, tokens, kv_heads):
    announce(f"kv write {tokens} tokens x {kv_heads} heads")
    rng = np.random.default_rng(tokens)
    k, v = (torch.from_numpy(rng.standard_normal((tokens, kv_heads, 128)).astype(np.float32)).to(torch.bfloat16)
            for _ in range(2))
    nb = (tokens + 15) // 16 + 1
    nb += 2
    ragged = np.arange(tokens) + 3 + 5 * (np.arange(tokens) // 37 % 2)       # prompts of 37 tokens, odd starts
    ragged = np.unique(ragged)[:tokens] if np.unique(ragged).size >= tokens else np.arange(tokens) + 1
    pairs = rng.permutation(nb * 8)[:(tokens + 1) // 2]                      # runs of two, aligned and not
    runs = (pairs[:, None] * 2 + np.array([0, 1])).reshape(-1)[:tokens]
    for slots in (np.arange(tokens) + 4, np.arange(tokens) + 3, rng.permutation(nb * 16)[:tokens], ragged, runs,
                  np.arange(tokens)[::-1] + 2):
        slots = slots.astype(np.int64)
        slots[tokens // 2] = -1 if tokens > 2 else slots[tokens // 2]
        write(fp8rl, k, v, slots, nb, 0.009, 0.011)
