"""GPU parity of the few-token GEMMs (at most 64 tokens, or a few rows per expert) against the fp64 oracle: every
tile's edges, fewer K blocks than waves, padded operands and outputs.  Pass criterion per element as in
test_gpu_gemm.py: |gpu - ref| <= 4e-3 |ref| + 1e-3 rms(ref) (bf16 rounding is 2^-9 of the value, the fp32 sums and
the instruction's truncation stay below the second term on these operands)."""
import numpy as np
import pytest
import torch

from oracle import cref, gemm
from tests.gpu_util import announce, bf16_to_f64, need_gpu, u16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp8rl():
    need_gpu()
    import paper_2601_18150_amd as m
    m.load()
    return m


def operands(rng, m, n, k):
    a = torch.from_numpy(rng.standard_normal((m, k)).astype(np.float32)).to(torch.bfloat16)
    w = torch.from_numpy((rng.standard_normal((n, k)) * 0.02).astype(np.float32)).to(torch.bfloat16)
    return (*cref.quant_act_token_group128(u16(a)), *cref.quant_weight_block128(u16(w)))


def pow2(s):
    return np.exp2(np.round(np.log2(s))).astype(np.float32)


def padded(x, cols, dtype):
    t = torch.zeros((x.shape[0], x.shape[1] + cols), dtype=dtype, device="cuda")
    t[:, :x.shape[1]] = torch.from_numpy(x).cuda()
    return t


def close(y, ref, what):
    ok, worst, _ = gemm.tolerance_check(bf16_to_f64(y), ref)
    assert ok, f"{what}: worst |err|/bound {worst:.3f}"


# N = 5120 and 5248 straddle the two weight-row tiles; K = 128 and 384 leave waves without a K block
@pytest.mark.parametrize("n,k", [(128, 128), (384, 384), (5120 - 128, 13 * 128), (5120, 13 * 128), (256, 96 * 128)])
@pytest.mark.parametrize("m", [1, 7, 8, 9, 16, 17, 32, 33, 63, 64])
def test_dense_few_tokens(fp8rl, m, n, k):
    announce(f"gemm few tokens m={m} n={n} k={k}")
    qa, sa, qw, sw = operands(np.random.default_rng(m * 7 + n + k), m, n, k)
    q, s, w = padded(qa, 48, torch.uint8)[:, :k], padded(sa[:, :m], 5, torch.float32), padded(qw, 16, torch.uint8)[:, :k]
    out = torch.full((m + 2, n + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    fp8rl.fp8rl_gemm_w8a8_block(q, s, w, torch.from_numpy(sw).cuda(), y=out[:m, :n])
    scratch = fp8rl.fp8rl_gemm_w8a8_block_noalloc(q, s, w, torch.from_numpy(sw).cuda())
    p_a, p_w = pow2(sa), pow2(sw)
    y2 = fp8rl.fp8rl_gemm_w8a8_block_ue8m0(q, padded(p_a[:, :m], 5, torch.float32), w, torch.from_numpy(p_w).cuda())
    torch.cuda.synchronize()
    close(out[:m, :n], gemm.gemm_ref_fp64(qa, sa, qw, sw), "fp32 scales")
    close(y2, gemm.gemm_ref_fp64(qa, p_a, qw, p_w), "power-of-two scales")
    assert torch.equal(scratch.view(torch.int16), out[:m, :n].contiguous().view(torch.int16))
    assert torch.all(out[m:] == 7.0) and torch.all(out[:, n:] == 7.0), "wrote outside y"


@pytest.mark.parametrize("n,k", [(128, 128), (384, 768), (256, 1152)])
@pytest.mark.parametrize("counts", [[1], [0, 0, 12, 0], [8, 9, 16, 17, 0, 0, 0, 0], [33, 0, 0, 1, 0, 0, 0],
                                    [170] + [0] * 14, [0] * 70 + [5, 3, 0, 31, 32]])
def test_grouped_few_rows(fp8rl, counts, n, k):
    """Experts with 0 .. 170 rows, at most 12 a expert on average: chunks of 8, 16 and 32 rows, several per workgroup."""
    announce(f"grouped gemm few rows {len(counts)} experts, {sum(counts)} rows, n={n} k={k}")
    rng = np.random.default_rng(sum(counts) + n + k)
    g, r, t = len(counts), sum(counts), 23
    assert r <= 12 * g
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    qt, st, qw, sw = operands(rng, t, g * n, k)
    qw, sw = qw.reshape(g, n, k), sw.reshape(g, n // 128, k // 128)
    index = rng.integers(0, t, r).astype(np.int32)
    qa, sa = np.ascontiguousarray(qt[index]), np.ascontiguousarray(st[:, index])
    w, s, off = torch.from_numpy(qw).cuda(), torch.from_numpy(sw).cuda(), torch.from_numpy(offsets).cuda()
    y = fp8rl.fp8rl_grouped_gemm_w8a8_block(torch.from_numpy(qa).cuda(), padded(sa, 3, torch.float32), w, s, off)
    yg = fp8rl.fp8rl_grouped_gemm_w8a8_block_gathered(padded(qt, 32, torch.uint8)[:, :k], padded(st, 1, torch.float32),
                                                      torch.from_numpy(index).cuda(), w, s, off)
    p_a, p_w = pow2(sa), pow2(sw)
    y2 = fp8rl.fp8rl_grouped_gemm_w8a8_block_ue8m0(torch.from_numpy(qa).cuda(), torch.from_numpy(p_a).cuda(), w,
                                                   torch.from_numpy(p_w).cuda(), off)
    torch.cuda.synchronize()
    close(y, gemm.grouped_gemm_ref_fp64(qa, sa, qw, sw, offsets), "fp32 scales")
    assert torch.equal(y.view(torch.int16), yg.view(torch.int16)), "gathered rows differ"
    close(y2, gemm.grouped_gemm_ref_fp64(qa, p_a, qw, p_w, offsets), "power-of-two scales")


def random_experts(rng, g, n, k, rows):
    """Operands without a quantiser: any finite E4M3 codes are valid ones (many experts, few rows)."""
    code = lambda *shape: (rng.integers(0, 0x7F, shape) | rng.integers(0, 2, shape) << 7).astype(np.uint8)
    scale = lambda *shape: np.exp2(rng.uniform(-9, -7, shape)).astype(np.float32)
    return code(rows, k), scale(k // 128, rows), code(g, n, k), scale(g, n // 128, k // 128)


# rows of some experts of G, the others have none: chunks of 128 rows with tails of 1, 8, 32, 33 and 128 rows beside
# chunks of 32; popular experts first, last and side by side; more than 256 experts (the four waves share the search)
@pytest.mark.parametrize("g,counts", [
    (24, {0: 288}), (24, {23: 264, 22: 24}), (48, {5: 257, 6: 256, 7: 33, 8: 1}), (48, {0: 161, 1: 384, 47: 31}),
    (256, {255: 700, 3: 289, 4: 1}), (257, {256: 650, 255: 64, 0: 33}), (300, {0: 1, 255: 130, 256: 300, 299: 97}),
    (1024, {1023: 900, 767: 417, 512: 256, 0: 32, 511: 33}), (1024, {}),
])
@pytest.mark.parametrize("n,k", [(128, 256), (256, 1152)])
def test_grouped_popular_experts(fp8rl, g, counts, n, k):
    announce(f"grouped gemm popular experts {counts} of {g}, n={n} k={k}")
    if g * n * k > 1 << 27:
        n = 128
    counts = counts or {e: 1 + (e % 7 == 0) * 40 for e in range(g)}
    rng = np.random.default_rng(g + sum(counts.values()) + k)
    c = np.zeros(g, np.int64)
    for e, rows in counts.items():
        c[e] = rows
    r = int(c.sum())
    assert r <= 12 * g, "the case is meant for the few-row kernel"
    offsets = np.concatenate([[0], np.cumsum(c)]).astype(np.int32)
    qt, st, qw, sw = random_experts(rng, g, n, k, 40)
    index = rng.integers(0, 40, r).astype(np.int32)
    qa, sa = np.ascontiguousarray(qt[index]), np.ascontiguousarray(st[:, index])
    w, s, off = torch.from_numpy(qw).cuda(), torch.from_numpy(sw).cuda(), torch.from_numpy(offsets).cuda()
    out = torch.full((r + 2, n), 7.0, dtype=torch.bfloat16, device="cuda")
    fp8rl.fp8rl_grouped_gemm_w8a8_block(torch.from_numpy(qa).cuda(), padded(sa, 3, torch.float32), w, s, off, y=out[:r])
    yg = fp8rl.fp8rl_grouped_gemm_w8a8_block_gathered(padded(qt, 32, torch.uint8)[:, :k], padded(st, 1, torch.float32),
                                                      torch.from_numpy(index).cuda(), w, s, off)
    p_a, p_w = pow2(sa), pow2(sw)
    y2 = fp8rl.fp8rl_grouped_gemm_w8a8_block_ue8m0(torch.from_numpy(qa).cuda(), torch.from_numpy(p_a).cuda(), w,
                                                   torch.from_numpy(p_w).cuda(), off)
    torch.cuda.synchronize()
    full = np.concatenate([[0], np.cumsum(c[c > 0])]).astype(np.int32)         # (the oracle needs no empty experts)
    close(out[:r], gemm.grouped_gemm_ref_fp64(qa, sa, qw[c > 0], sw[c > 0], full), "fp32 scales")
    assert torch.equal(out[:r].view(torch.int16), yg.view(torch.int16)), "gathered rows differ"
    close(y2, gemm.grouped_gemm_ref_fp64(qa, p_a, qw[c > 0], p_w[c > 0], full), "power-of-two scales")
    assert torch.all(out[r:] == 7.0), "wrote outside y"


def test_one_expert_with_all_rows_is_no_serial_chain(fp8rl):
    """3072 rows of 256 experts: all in one expert read 1/256 of the weights, so the call may not take as long as with
    12 rows in each (measured 0.23 of it; 1.14 when a few workgroups walked the expert's rows)."""
    announce("grouped gemm: one expert with all the rows, timed")
    g, n, k, rows = 256, 2048, 768, 3072
    gen = torch.Generator(device="cuda").manual_seed(1)
    codes = lambda *shape: torch.randint(0, 120, shape, dtype=torch.uint8, device="cuda", generator=gen)
    qa, qw = codes(rows, k), codes(g, n, k)
    sa, sw = torch.ones((k // 128, rows), device="cuda"), torch.ones((g, n // 128, k // 128), device="cuda")
    y = torch.empty((rows, n), dtype=torch.bfloat16, device="cuda")

    def span(counts):
        off = torch.tensor([0] + torch.tensor(counts).cumsum(0).tolist(), dtype=torch.int32, device="cuda")
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                fp8rl.fp8rl_grouped_gemm_w8a8_block(qa, sa, qw, sw, off, y=y)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 20)
        return sorted(times)[3]

    even, one = span([rows // g] * g), span([0] * 99 + [rows] + [0] * (g - 100))
    assert one < 0.6 * even, f"one expert {one * 1e3:.1f} us, spread evenly {even * 1e3:.1f} us"
