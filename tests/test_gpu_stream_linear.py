"""The streaming linear kernel (a handful of rows): edges of its row tiles, column remainders, K tails, every epilogue,
against the CPU oracle; and the same bits for a row whatever the rows batched with it."""
import numpy as np
import pytest
import torch

import synth
from oracle import sfo

from gpu_common import dev, engine_only, rel_err, to_np

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2      # bf16 results against the fp64 oracle (max |diff| / max |ref|)


def engine():
    return engine_only(synth.ModelShape("t", 1, 128, 2, 2, 64, 256, 512, "bf16"), 1, 64, 1)


def operands(M, N, K, seed):
    g = synth.rng(seed, M * 7919 + N * 31 + K)
    x = synth.to_bf16_values(g.standard_normal((M, K), dtype=np.float32))
    w = synth.to_bf16_values(g.standard_normal((N, K), dtype=np.float32) * 0.05)
    return g, x, w


# rows: 1, around 8 (the K rule) and 16 (one or two row tiles), 32; columns: 16 and 32 per workgroup with remainders of
# 8 and 24; K: less than one chunk, a tail of 8, an odd number of 16-steps, fewer chunks than waves, many batches.
# fp32 accumulators of K <= 2600 bf16 products: 1e-5 of the largest result (as for the tiled kernel).
@pytest.mark.parametrize("M", [1, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("N,K", [(8, 8), (136, 264), (4104, 112), (56, 2600)])
def test_stream_linear(M, N, K):
    g, x, w = operands(M, N, K, 41)
    bias = synth.to_bf16_values(g.standard_normal(N, dtype=np.float32))
    res = synth.to_bf16_values(g.standard_normal((M, N), dtype=np.float32))
    eng = engine()
    ref = sfo.linear(x, w)
    xd, wd = dev(x, "bf16"), dev(w, "bf16")
    packed = (eng.sf_pack_weight(wd), N)
    y = eng.sf_op_linear(xd, None, out_f32=True, packed=packed)
    assert rel_err(to_np(y), ref) < 1e-5
    r = dev(res, "bf16")                     # bias, residual aliasing the output
    eng.sf_op_linear(xd, None, bias=dev(bias, "bf16"), residual=r, y=r, packed=packed)
    assert rel_err(to_np(r), ref + bias + res) < BF16_TOL


@pytest.mark.parametrize("M", [3, 16, 30])
@pytest.mark.parametrize("F,K", [(32, 136), (224, 1000)])
def test_stream_norm_and_gate(M, F, K):
    g, x, w = operands(M, 2 * F, K, 43)
    x[0] *= 40.0
    x = synth.to_bf16_values(x)
    gain = synth.to_bf16_values(1.0 + 0.5 * g.standard_normal(K, dtype=np.float32))
    eng = engine()
    xd, wd, gd = dev(x, "bf16"), dev(w, "bf16"), dev(gain, "bf16")
    y = eng.sf_op_rmsnorm_linear(xd, gd, wd, out_f32=True)
    assert rel_err(to_np(y), sfo.linear(sfo.rmsnorm(x, gain, 1e-6), w)) < 5e-3   # weight * gain is rounded to bf16 once
    one = eng.sf_op_rmsnorm_linear(xd[:1].contiguous(), gd, wd, out_f32=True)
    torch.cuda.synchronize()
    assert torch.equal(one, y[:1])           # one row tile or two: a row's sums are the same
    xs = synth.to_bf16_values(x * 0.1)
    gu = sfo.linear(xs, w)
    act = eng.sf_op_linear_swiglu(dev(xs, "bf16"), wd)
    assert rel_err(to_np(act), sfo.silu_mul(gu[:, :F], gu[:, F:])) < BF16_TOL
