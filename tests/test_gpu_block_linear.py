"""The block kernel (both operands through LDS by direct loads): edges of its row and column tiles, fewer K slices than it
keeps in flight, every epilogue, against the CPU oracle; and the ring kernel's bits."""
import numpy as np
import pytest
import torch

import synth
from oracle import sfo

from paper_2511_20340_amd import binding as sfb
from paper_2511_20340_amd.engine import Engine

from gpu_common import dev, engine_only, linear_choice, rel_err, to_np

pytestmark = pytest.mark.gpu

BLOCK_TILES = range(15, 26)
RING_TILE = 2


def block_runs(tile, M, N, K, split, flags=0):
    """Whether the forced tile runs (a tile that cannot take the layer is replaced by a ring tile): the tiles with groups of
    waves take layers whose K is cut into as many parts, the narrow ones no arg-max."""
    kernel, runs, _ = linear_choice(M, N, K, flags, tile=tile, split=split)
    slices = -(-K // 64)
    parts = -(-slices // -(-slices // min(split, slices)))
    takes = {23: 2, 24: 4, 25: 2}.get(tile, parts) == parts and not (flags & sfb.SF_LINEAR_ARGMAX and tile >= 19 and tile != 22)
    assert (kernel, runs) == ((sfb.SF_KERNEL_BLOCK, tile) if takes else (sfb.SF_KERNEL_RING, 10)), (tile, split)
    return takes


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
                if block_runs(tile, M, N, K, split):
                    for got, w_ in zip(outputs(tile, split), want):
                        assert torch.equal(got, w_), (tile, split)
    finally:
        eng.sf_tune_linear(0, 0)


@pytest.mark.parametrize("M,N,K", [(97, 1032, 192), (330, 520, 64)])
def test_block_argmax(M, N, K):
    """Arg-max partials (integer operands: exact, ties everywhere) through every tile that forms them."""
    g = synth.rng(53, M + N)
    x = g.integers(-2, 3, (M, K)).astype(np.float32)
    w = g.integers(-1, 2, (N, K)).astype(np.float32)
    eng = engine()
    xd, wd = dev(x, "bf16"), dev(w, "bf16")
    want = sfo.linear(x, w).argmax(-1)
    ran = []
    try:
        for tile in (RING_TILE, *BLOCK_TILES):
            if tile == RING_TILE or block_runs(tile, M, N, K, 1, sfb.SF_LINEAR_ARGMAX):
                eng.sf_tune_linear(tile, 1)
                np.testing.assert_array_equal(eng.sf_op_linear_argmax(xd, wd).cpu().numpy(), want, err_msg=f"tile {tile}")
                ran.append(tile)
    finally:
        eng.sf_tune_linear(0, 0)
    assert ran == [RING_TILE, 15, 16, 17, 18, 22]


@pytest.mark.parametrize("M,F,K", [(97, 160, 192), (330, 288, 64), (70, 96, 512), (161, 160, 320)])
def test_block_gate(M, F, K):
    """The SwiGLU gate through every tile, unsplit and split: in the workgroup, between its groups of waves, and in the second
    launch behind ring and block tiles."""
    g = synth.rng(54, M + F)
    x = synth.to_bf16_values(g.standard_normal((M, K), dtype=np.float32))
    wgu = synth.to_bf16_values(g.standard_normal((2 * F, K), dtype=np.float32) * 0.05)
    gu = sfo.linear(x, wgu)
    ref = sfo.silu_mul(gu[:, :F], gu[:, F:])
    eng = engine()
    xd, wd = dev(x, "bf16"), dev(wgu, "bf16")
    try:
        for split in (1, 2, 4):
            eng.sf_tune_linear(RING_TILE, split)
            want = eng.sf_op_linear_swiglu(xd, wd).clone()
            assert rel_err(to_np(want), ref) < 2e-2        # bf16 results against the fp64 oracle, as in the other tests
            for tile in BLOCK_TILES:
                if block_runs(tile, M, 2 * F, K, split, sfb.SF_LINEAR_GLU):
                    eng.sf_tune_linear(tile, split)
                    assert torch.equal(eng.sf_op_linear_swiglu(xd, wd), want), (tile, split)
    finally:
        eng.sf_tune_linear(0, 0)


@pytest.mark.parametrize("split", [1, 2, 4])
def test_block_gate_with_the_norm(split):
    """Gate and up projection as a step runs them, with the fused norm, every layer of the step forced onto each tile."""
    shape, B, k, cap = synth.ModelShape("t", 1, 512, 4, 2, 128, 640, 1032, "bf16"), 15, 4, 64
    weights = synth.target_weights(shape, 3, 0.05)
    g = synth.rng(55, split)
    toks = g.integers(0, shape.vocab, (B, k + 1)).astype(np.int32)
    eng = Engine(shape.cfg(), B, cap, k)
    eng.bind(weights, None)

    def step(tile):
        eng.sf_tune_linear(tile, split)
        eng.set_state(kv_len=np.full(B, 2, np.int32), pending=toks[:, 0], n_new=np.ones(B, np.int32))
        logits, ids = eng.sf_verify_step(k, torch.from_numpy(toks[:, 1:].copy()).cuda())
        torch.cuda.synchronize()
        return logits.clone(), ids.clone(), eng.hooks.clone(), eng.sf_kv_export("tk", 0), eng.sf_kv_export("tv", 0)
    try:
        want, ran = step(RING_TILE), 0
        for tile in BLOCK_TILES:
            if block_runs(tile, B * (k + 1), 2 * shape.d_ffn, shape.d_model, split, sfb.SF_LINEAR_GLU | sfb.SF_LINEAR_NORM):
                ran += 1
                assert block_runs(tile, B * (k + 1), shape.d_model, shape.d_ffn, split)      # the down projection too
                for got, ref in zip(step(tile), want):
                    assert torch.equal(got, ref), tile
    finally:
        eng.sf_tune_linear(0, 0)
    assert ran == {1: 8, 2: 10, 4: 9}[split]
