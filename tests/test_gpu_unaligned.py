"""Linear layers whose output, residual and bias do not start on 16 bytes leave and fetch element by element: the same bits
as through the 16-byte units, in every kernel that has the epilogue, and nothing outside the rows."""
import numpy as np
import pytest
import torch

import synth
from paper_2511_20340_amd import binding as sfb

from gpu_common import dev, engine_only, linear_choice

pytestmark = pytest.mark.gpu

RING, BLOCK, STREAM = sfb.SF_KERNEL_RING, sfb.SF_KERNEL_BLOCK, sfb.SF_KERNEL_STREAM


def off_by_one(shape, dtype, fill=None):
    """A tensor one element behind a 16-byte boundary, and the buffer around it."""
    n = int(np.prod(shape))
    room = torch.full((n + 16,), 777.0, dtype=dtype, device="cuda")
    t = room[1:1 + n].view(shape)
    assert room.data_ptr() % 16 == 0
    if fill is not None:
        t.copy_(fill)
    return t, room


# (forced tile, split) -> what runs: the ring kernel with one and five 32x32 tiles a wave, split with its second launch, the
# tallest tile; the block kernel with 2 x 4 waves, split, and with groups of waves that share K; the streaming kernel
@pytest.mark.parametrize("M,N,K,tile,split,kernel", [
    (40, 264, 128, 1, 1, RING), (170, 264, 128, 10, 1, RING), (330, 264, 128, 11, 1, RING), (40, 264, 512, 2, 2, RING),
    (130, 264, 128, 18, 1, BLOCK), (130, 264, 512, 16, 4, BLOCK), (70, 264, 512, 23, 2, BLOCK), (70, 264, 512, 24, 4, BLOCK),
    (5, 264, 264, 0, 0, STREAM), (30, 264, 2072, 0, 0, STREAM)])
@pytest.mark.parametrize("out_f32", [False, True])
def test_unaligned_output_residual_and_bias(M, N, K, tile, split, kernel, out_f32):
    assert linear_choice(M, N, K, tile=tile, split=split)[0] == kernel
    eng = engine_only(synth.ModelShape("t", 1, 128, 2, 2, 64, 256, 512, "bf16"), 1, 64, 1)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    x, packed = rand(M, K), (eng.sf_pack_weight(rand(N, K)), N)
    bias, res = rand(N), rand(M, N)
    dtype = torch.float32 if out_f32 else torch.bfloat16
    eng.sf_tune_linear(tile, split)
    try:
        want = eng.sf_op_linear(x, None, bias=bias, residual=res, out_f32=out_f32, packed=packed)
        y, room = off_by_one((M, N), dtype)
        b1, r1 = off_by_one((N,), torch.bfloat16, bias)[0], off_by_one((M, N), torch.bfloat16, res)[0]
        eng.sf_op_linear(x, None, bias=b1, residual=r1, out_f32=out_f32, y=y, packed=packed)
        assert torch.equal(y, want)
        assert room[0] == 777.0 and bool((room[1 + M * N:] == 777.0).all())
        for one in (dict(bias=b1, residual=res), dict(bias=bias, residual=r1)):      # any one of them is enough
            assert torch.equal(eng.sf_op_linear(x, None, out_f32=out_f32, packed=packed, **one), want)
    finally:
        eng.sf_tune_linear(0, 0)


# the gate is the one operation that takes rows at any address: the block kernel's direct loads move 16 bytes from where
# they start on 16, so such rows go to the ring kernel
@pytest.mark.parametrize("M,F,K", [(5, 96, 264), (130, 288, 128), (330, 1056, 128), (160, 2048, 4096)])
def test_unaligned_rows_of_the_gate(M, F, K):
    unaligned = linear_choice(M, 2 * F, K, sfb.SF_LINEAR_GLU | sfb.SF_LINEAR_UNALIGNED)
    aligned = linear_choice(M, 2 * F, K, sfb.SF_LINEAR_GLU)
    assert unaligned[0] != BLOCK and unaligned[2] == aligned[2] and (M <= 32) == (aligned[0] == STREAM)
    eng = engine_only(synth.ModelShape("t", 1, 128, 2, 2, 64, 256, 512, "bf16"), 1, 64, 1)
    g = torch.Generator(device="cuda").manual_seed(M + F)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    w = (torch.randn(2 * F, K, generator=g, device="cuda") * 0.05).bfloat16()
    want = eng.sf_op_linear_swiglu(x, w).clone()
    assert torch.equal(eng.sf_op_linear_swiglu(off_by_one((M, K), torch.bfloat16, x)[0], w), want)
