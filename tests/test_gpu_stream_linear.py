"""The streaming linear kernel (a handful of rows): edges of its row tiles, column remainders, K tails, every epilogue,
against the CPU oracle; and the ring kernel's bits at the same split."""
import numpy as np
import pytest
import torch

import synth
from oracle import sfo

from gpu_common import dev, engine_only, linear_choice, rel_err, to_np
from paper_2511_20340_amd import binding as sfb

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2      # bf16 results against the fp64 oracle (max |diff| / max |ref|)


def engine():
    return engine_only(synth.ModelShape("t", 1, 128, 2, 2, 64, 256, 512, "bf16"), 1, 64, 1)


def operands(M, N, K, seed):
    g = synth.rng(seed, M * 7919 + N * 31 + K)
    x = synth.to_bf16_values(g.standard_normal((M, K), dtype=np.float32))
    w = synth.to_bf16_values(g.standard_normal((N, K), dtype=np.float32) * 0.05)
    return g, x, w


# rows: 1, around 8, around 16 (one or two row tiles), 32; columns: remainders of 8; K: less than one chunk, a tail of 8, an
# odd number of 16-steps, 4 parts of uneven length.
# fp32 accumulators of K <= 2600 bf16 products: 1e-5 of the largest result (as for the tiled kernel).
@pytest.mark.parametrize("M", [1, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("N,K", [(8, 8), (136, 264), (4104, 112), (56, 2600)])
def test_stream_linear(M, N, K):
    g, x, w = operands(M, N, K, 41)
    bias = synth.to_bf16_values(g.standard_normal(N, dtype=np.float32))
    res = synth.to_bf16_values(g.standard_normal((M, N), dtype=np.float32))
    eng = engine()
    assert linear_choice(M, N, K)[0] == sfb.SF_KERNEL_STREAM
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
    assert linear_choice(M, 2 * F, K, sfb.SF_LINEAR_NORM)[0] == linear_choice(M, 2 * F, K, sfb.SF_LINEAR_GLU)[0] == sfb.SF_KERNEL_STREAM
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


def with_ring(eng, split, call):
    eng.sf_tune_linear(1, split)
    try:
        return call()
    finally:
        eng.sf_tune_linear(0, 0)


# (split, 16-column tiles per wave) in all combinations; remainders of 8 columns; K that ends 8, 16 and 24 positions into a
# chunk; parts of uneven length (41, 33 and 65 slices); the rows of one and two tiles, and of several row tiles
@pytest.mark.parametrize("N,K,want,rows", [
    (136, 264, (1, 1), (1, 16, 17, 32)), (16392, 264, (1, 2), (5, 32)), (72, 1032, (2, 1), (1, 16, 17, 32)),
    (8200, 1048, (2, 2), (5, 32)), (264, 2072, (4, 1), (1, 16, 17, 32)), (56, 2600, (4, 1), (16, 32)),
    (4104, 2064, (4, 2), (5, 32)), (136, 4104, (8, 1), (1, 16, 17)), (72, 1000, (2, 1), (33, 64, 97)),
    (136, 2040, (4, 1), (33, 97)), (2504, 2048, (4, 2), (33, 64))])
def test_stream_gives_the_split_kernels_bits(N, K, want, rows):
    """Plain, fused norm, bias + residual in place: as the ring kernel with that split (and its second launch)."""
    eng = engine()
    for M in rows:
        g, x, w = operands(M, N, K, 51)
        gain = synth.to_bf16_values(1.0 + 0.5 * g.standard_normal(K, dtype=np.float32))
        xd, wd, gd = dev(x, "bf16"), dev(w, "bf16"), dev(gain, "bf16")
        bias = dev(g.standard_normal(N, dtype=np.float32), "bf16")
        res = dev(g.standard_normal((M, N), dtype=np.float32), "bf16")
        kernel, tiles, split = linear_choice(M, N, K)
        assert (kernel, split, tiles) == (sfb.SF_KERNEL_STREAM, *want), M
        plain, folded = (eng.sf_pack_weight(wd), N), (eng.sf_pack_weight(wd, gain=gd), N)

        def outputs():
            r = res.clone()
            eng.sf_op_linear(xd, None, bias=bias, residual=r, y=r, packed=plain)
            return r, eng.sf_op_linear(xd, None, out_f32=True, packed=plain), eng.sf_op_rmsnorm_linear(xd, gd, None, out_f32=True, packed=folded)
        for got, ref in zip(outputs(), with_ring(eng, split, outputs)):
            assert torch.equal(got, ref), M


@pytest.mark.parametrize("F,K,want,rows", [(32, 136, (1, 1), (1, 17)), (8224, 264, (1, 2), (3,)), (224, 1000, (2, 1), (16, 30, 70)),
                                           (4128, 1032, (2, 2), (17,)), (32, 2056, (4, 2), (3, 30)), (288, 4104, (8, 2), (1, 3))])
def test_stream_gate_gives_the_split_kernels_bits(F, K, want, rows):
    eng = engine()
    for M in rows:
        _, x, w = operands(M, 2 * F, K, 52)
        xd, wd = dev(x, "bf16"), dev(w, "bf16")
        kernel, tiles, split = linear_choice(M, 2 * F, K, sfb.SF_LINEAR_GLU)
        assert (kernel, split, tiles) == (sfb.SF_KERNEL_STREAM, *want), M
        gate = lambda: eng.sf_op_linear_swiglu(xd, wd).clone()
        assert torch.equal(gate(), with_ring(eng, split, gate)), M


@pytest.mark.parametrize("M,N,K", [(5, 72, 264), (17, 56, 2600), (5, 136, 4104), (40, 72, 1000)])
def test_stream_infinite_weight_stays_in_its_column(M, N, K):
    """An infinite weight gives an infinity in its own column; it must not meet the zeros that stand for K positions outside
    a part (or outside K), which would make a NaN of it."""
    g, x, w = operands(M, N, K, 53)
    x = np.abs(x) + 0.5
    at = {8 * i: k for i, k in enumerate((0, K // 2, K - 1, K - 9, K // 4 + 3, K // 8))}
    for n, k in at.items():
        w[n, k] = np.inf
    assert linear_choice(M, N, K)[0] == sfb.SF_KERNEL_STREAM
    y = to_np(engine().sf_op_linear(dev(x, "bf16"), dev(w, "bf16"), out_f32=True))
    cols = np.array(sorted(at))
    assert np.all(y[:, cols] == np.inf) and np.all(np.isfinite(np.delete(y, cols, 1)))
