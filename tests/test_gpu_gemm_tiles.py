"""The dense GEMM across its tile choices (64x64 to 256x256, one tile per workgroup and persistent): ragged last
tiles in both directions, fewer K blocks than ring slots, odd K block counts (uneven wave groups), padded operands.
Pass criterion per element as in test_gpu_gemm.py."""
import numpy as np
import pytest
import torch

from oracle import gemm
from tests.gpu_util import announce, need_gpu
from tests.test_gpu_gemm_small import close, operands, padded, pow2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp8rl():
    need_gpu()
    import paper_2601_18150_amd as m
    m.load()
    return m


# (which tile a shape runs on is checked on the host, test_host_gemm_plan.py)
TILE_CASES = {
    # up to four K blocks (and above, where K = 5 * 128)
    "64x64-short": [(65, 128, 128), (100, 256, 384), (65, 128, 512), (257, 640, 256), (129, 2688, 384)],   # one wave group
    "persistent": [(1400, 12800, 256), (200, 24576, 512), (6355, 640, 128), (1570, 12160, 5 * 128)],       # 128x128
    "256x256": [(2100, 6272, 384), (1300, 6272, 5 * 128), (300, 24704, 5 * 128), (2100, 6144, 1024)],      # last tile of 128
    # above (two wave groups split K in the first three)
    "64x64": [(65, 128, 5 * 128), (129, 1024, 13 * 128), (256, 4096, 9 * 128)],
    "64x128": [(300, 4096, 5 * 128), (512, 4096, 5 * 128), (257, 5120, 7 * 128)],
    "128x64": [(300, 6144, 6 * 128), (257, 5632, 13 * 128)],
    "128x128": [(777, 4096, 5 * 128), (1000, 4096, 6 * 128)],                                              # eight waves
    "128x256": [(200, 24576, 5 * 128), (777, 6272, 6 * 128)],
    "256x128": [(640, 24704, 5 * 128), (600, 24576, 6 * 128)],                                             # last tile of 128
    "two launches": [(777, 24576, 9 * 128), (3001, 6272, 7 * 128), (1400, 12800, 5 * 128)],                # columns
}


@pytest.mark.parametrize("m,n,k", [shape for shapes in TILE_CASES.values() for shape in shapes])
def test_dense_tile_choices(fp8rl, m, n, k):
    announce(f"gemm tiles m={m} n={n} k={k}")
    qa, sa, qw, sw = operands(np.random.default_rng(m + n + k), m, n, k)
    q, s, w = padded(qa, 48, torch.uint8)[:, :k], padded(sa[:, :m], 5, torch.float32), padded(qw, 16, torch.uint8)[:, :k]
    sw_d = torch.from_numpy(sw).cuda()
    out = torch.full((m + 1, n + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    fp8rl.fp8rl_gemm_w8a8_block(q, s, w, sw_d, y=out[:m, :n])
    again = fp8rl.fp8rl_gemm_w8a8_block(q, s, w, sw_d)
    torch.cuda.synchronize()
    close(out[:m, :n], gemm.gemm_ref_fp64(qa, sa, qw, sw), "fp32 scales")
    assert torch.equal(again.view(torch.int16), out[:m, :n].contiguous().view(torch.int16)), "not deterministic"
    assert torch.all(out[m:] == 7.0) and torch.all(out[:, n:] == 7.0), "wrote outside y"
    p_a, p_w = pow2(sa), pow2(sw)
    y2 = fp8rl.fp8rl_gemm_w8a8_block_ue8m0(q, padded(p_a[:, :m], 5, torch.float32), w, torch.from_numpy(p_w).cuda())
    torch.cuda.synchronize()
    close(y2, gemm.gemm_ref_fp64(qa, p_a, qw, p_w), "power-of-two scales")
