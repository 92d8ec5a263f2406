"""The block kernel (both operands through LDS by direct loads): edges of its row and column tiles, fewer K slices than it
keeps in flight, every epilogue, against the CPU oracle; and the ring kernel's bits."""
import numpy as np
import pytest
import torch

import synth
from oracle import sfo

from gpu_common import dev, engine_only, rel_err, to_np

pytestmark = pytest.mark.gpu

BLOCK_TILES = range(15, 26)
RING_TILE = 2


def engine():
    return engine_only(synth.ModelShape("t", 1, 128, 2, 2, 64, 256, 512, "bf16"), 1, 64, 1)


# rows: one, around the 32-row blocks, around the tallest tile; columns: a remainder of 8 behind 32, 64 and 256; K: one slice
# (every load past it repeats the last), one more than the two to five slices in LDS, a split that leaves slices uneven.
# fp32 accumulators of K <= 704 bf16 products: 1e-5 of the largest result, as for the other kernels.
@pytest.mark.parametrize("M", [1, 33, 160, 321])
@pytest.mark.parametrize("N,K", [(8, 64), (40, 128), (72, 384), (264, 704)])
def test_block_linear(M, N, K):
    g = synth.rng(47, M * 7919 + N * 31 + K)
    x = synth.to_bf16_values(g.standard_normal((M, K), dtype=np.float32))
    w = synth.to_bf16_values(g.standard_normal((N, K), dtype=np.float32) * 0.05)
    gain = synth.to_bf16_values(1.0 + 0.5 * g.standard_normal(K, dtype=np.float32))
    bias = synth.to_bf16_values(g.standard_normal(N, dtype=np.float32))
    res = synth.to_bf16_values(g.standard_normal((M, N), dtype=np.float32))
    ref, ref_norm = sfo.linear(x, w), sfo.linear(sfo.rmsnorm(x, gain, 1e-6), w)
    eng = engine()
    xd, wd, gd, bd = dev(x, "bf16"), dev(w, "bf16"), dev(gain, "bf16"), dev(bias, "bf16")
    plain, folded = (eng.sf_pack_weight(wd), N), (eng.sf_pack_weight(wd, gain=gd), N)

    def outputs(tile, split):
        eng.sf_tune_linear(tile, split)
        r = dev(res, "bf16")                 # bias, residual aliasing the output
        eng.sf_op_linear(xd, None, bias=bd, residual=r, y=r, packed=plain)
        y = eng.sf_op_linear(xd, None, out_f32=True, packed=plain)
        return y, r, eng.sf_op_rmsnorm_linear(xd, gd, None, out_f32=True, packed=folded)
    try:
        for split in (1, 2, 3, 4):
            want = [t.clone() for t in outputs(RING_TILE, split)]
            assert rel_err(to_np(want[0]), ref) < 1e-5
            assert rel_err(to_np(want[2]), ref_norm) < 5e-3     # weight * gain is rounded to bf16 once
            for tile in BLOCK_TILES:
                for got, w_ in zip(outputs(tile, split), want):
                    assert torch.equal(got, w_), (tile, split)
    finally:
        eng.sf_tune_linear(0, 0)


@pytest.mark.parametrize("M,N,K,F", [(97, 1032, 192, 160), (330, 520, 64, 288)])
def test_block_argmax_and_gate(M, N, K, F):
    """Arg-max partials (integer operands: exact, ties everywhere) and the SwiGLU gate through every tile."""
    g = synth.rng(53, M + N)
    x = g.integers(-2, 3, (M, K)).astype(np.float32)
    w = g.integers(-1, 2, (N, K)).astype(np.float32)
    wgu = synth.to_bf16_values(g.standard_normal((2 * F, K), dtype=np.float32) * 0.05)
    eng = engine()
    xd, wd, wgud = dev(x, "bf16"), dev(w, "bf16"), dev(wgu, "bf16")
    want = sfo.linear(x, w).argmax(-1)
    try:
        first = None
        for tile in (RING_TILE, *BLOCK_TILES):
            eng.sf_tune_linear(tile, 1)
            ids = eng.sf_op_linear_argmax(xd, wd)
            np.testing.assert_array_equal(ids.cpu().numpy(), want, err_msg=f"tile {tile}")
            act = eng.sf_op_linear_swiglu(xd, wgud)
            first = act.clone() if first is None else first
            assert torch.equal(act, first), tile
    finally:
        eng.sf_tune_linear(0, 0)
