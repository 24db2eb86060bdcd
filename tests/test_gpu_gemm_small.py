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
