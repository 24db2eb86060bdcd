"""Decode attention where its split of the work changes: one split and many, waves with no page, a last page of one
token, two and more records per sequence, both cache types.  Tolerance as in test_gpu_kv.py."""
import numpy as np
import pytest
import torch

from oracle import gemm, kv
from tests.gpu_util import announce, need_gpu, u16
from tests.test_gpu_kv import paged_inputs, run_fp8

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp8rl():
    need_gpu()
    import paper_2601_18150_amd as m
    m.load()
    return m


# pages per split: 16 up to 256 tokens (one record, written by the attention kernel itself), then several records;
# (160, ..): more workgroups than are resident; (1, 3): few, long sequences
@pytest.mark.parametrize("batch,q_heads,kv_heads,max_len", [(5, 8, 1, 256), (5, 8, 1, 257), (3, 4, 4, 1025),
                                                           (1, 8, 1, 9000), (160, 16, 8, 520)])
def test_attention_split_edges(fp8rl, batch, q_heads, kv_heads, max_len):
    announce(f"attention splits batch={batch} heads={q_heads}/{kv_heads} max_len={max_len}")
    rng = np.random.default_rng(batch * 100 + max_len)
    lens = rng.integers(0, max_len + 1, batch).astype(np.int32)
    lens[:3] = [max_len, 1, min(max_len, 33)][:len(lens[:3])]
    q, kc, vc, table, _ = paged_inputs(rng, lens, q_heads, kv_heads)
    ks, vs, sm = np.float32(0.02), np.float32(0.03), float(1 / np.sqrt(128))
    out = run_fp8(fp8rl, q, kc, vc, table, lens, ks, vs, sm, max_seq_len=max_len)
    again = run_fp8(fp8rl, q, kc, vc, table, lens, ks, vs, sm, max_seq_len=max_len)
    ref = kv.attention_decode(u16(q), kc, vc, ks, vs, table, lens, sm)
    ok, worst, _ = gemm.tolerance_check(out.float().cpu().numpy().astype(np.float64).reshape(ref.shape), ref)
    assert ok, f"worst |err|/bound {worst:.3f}"
    assert torch.equal(out.view(torch.int16), again.view(torch.int16)), "not deterministic"
    assert torch.all(out[torch.from_numpy(lens == 0)] == 0)


# a split is 16 pages, wave w of it starts at page w: its first page, all first pages, a whole split, all but one token
@pytest.mark.parametrize("max_len", [256, 1025])
@pytest.mark.parametrize("pages", [[0], [1], [0, 1, 2, 3], list(range(16)), [5, 6, 15]])
def test_scores_past_the_range_of_fp32_weigh_nothing(fp8rl, pages, max_len):
    """Whole pages whose scores overflow to -inf have weight 0 wherever they stand, as one such token among others has
    (the fp64 oracle's scores do not overflow; their weights underflow to 0)."""
    announce(f"attention -inf scores in pages {pages}, max_len={max_len}")
    rng = np.random.default_rng(max_len + len(pages))
    lens = np.array([max_len, max_len - 5], np.int32)
    q, kc, vc, table, _ = paged_inputs(rng, lens, 8, 2)
    q[:, :, 0] = 3.0e38
    kc[..., 0] = 0                                    # elsewhere: the other 127 dims decide
    for b in range(len(lens)):
        for p in pages:
            kc[table[b, p], :, :, 0] = 0xFE           # -448
        if max_len == 256 and len(pages) == 16:
            kc[table[b, 7], :, 3, 0] = 0              # (one token keeps a finite score)
    ks, vs, sm = np.float32(0.02), np.float32(0.03), float(1 / np.sqrt(128))
    out = run_fp8(fp8rl, q, kc, vc, table, lens, ks, vs, sm, max_seq_len=max_len)
    ref = kv.attention_decode(u16(q), kc, vc, ks, vs, table, lens, sm)
    ok, worst, _ = gemm.tolerance_check(out.float().cpu().numpy().astype(np.float64).reshape(ref.shape), ref)
    assert ok, f"worst |err|/bound {worst:.3f}"


@pytest.mark.parametrize("gap", [-48.0, -60.0, -72.0])
def test_partial_results_are_combined_in_full_fp32(fp8rl, gap):
    """One wave of a split scores 0, the other three score `gap` and hold all the value: their 192 tokens' sum in the
    split's record (fp32, behind the o[128] of the one head: its maximum) is 192 e^gap within 5e-7, two roundings of
    the weight's ulp and two of the sum; an exponential by a rounded gap * log2(e) is off by 2 to 3e-6 here."""
    announce(f"attention: combination of the waves, gap {gap}")
    n = 512                                           # two splits of 16 pages, wave w attends over pages w, w + 4, ...
    kc, vc = torch.zeros((32, 1, 16, 128)), torch.ones((32, 1, 4, 128, 4))
    first = torch.arange(32) % 4 == 0
    kc[~first, :, :, 0] = gap                         # (exact in E4M3)
    vc[first] = 0
    kc, vc = (x.to(torch.float8_e4m3fn).view(torch.uint8).cuda() for x in (kc, vc))
    q = torch.zeros((1, 1, 128), dtype=torch.bfloat16)
    q[..., 0] = 1.0
    table = torch.arange(32, dtype=torch.int32).reshape(1, 32)
    one = torch.ones(1, dtype=torch.float32, device="cuda")
    need = fp8rl.fp8rl_attention_decode_workspace_size(1, 1, 1, n)
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    fp8rl.fp8rl_attention_decode_fp8kv(q.cuda(), kc, vc, table.cuda(),
                                       torch.tensor([n], dtype=torch.int32, device="cuda"), n, one, one, 1.0, workspace=ws)
    torch.cuda.synchronize()
    rec = ws.cpu().double().reshape(2, -1)[:, :129].numpy()
    assert np.all(rec[:, 128] == 0.0), "the records' maxima"
    assert np.all(np.abs(rec[:, :128] / (192 * np.exp(gap)) - 1) < 5e-7), rec[:, 0] / (192 * np.exp(gap)) - 1
