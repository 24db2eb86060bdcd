"""The Python entry points refuse wrong arguments with the exception that names the fault, before they ask for a
stream: the same on a machine without a GPU."""
import pytest
import torch

import paper_2601_18150_amd as fp8rl


def linear_args(dtype=torch.bfloat16):
    return torch.zeros((4, 128), dtype=dtype), torch.zeros((128, 128), dtype=torch.uint8), torch.ones((1, 1))


def test_linear_on_host_tensors():
    with pytest.raises(ValueError, match="HIP device"):
        fp8rl.linear_w8a8(*linear_args())


def test_linear_of_another_dtype():
    with pytest.raises(TypeError):
        fp8rl.linear_w8a8(*linear_args(torch.float32))


@pytest.mark.parametrize("call", [
    lambda x, q, sa, sw: fp8rl.fp8rl_quant_act_token_group128(x),
    lambda x, q, sa, sw: fp8rl.fp8rl_gemm_w8a8_block(q[:4], sa, q, sw),
    lambda x, q, sa, sw: fp8rl.fp8rl_gemm_w8a8_block_noalloc(q[:4], sa, q, sw),
])
def test_steps_on_host_tensors(call):
    x, q, sw = linear_args()
    with pytest.raises(ValueError, match="HIP device"):
        call(x, q, torch.ones((1, 4)), sw)
