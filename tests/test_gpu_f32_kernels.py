"""fp32 mode: the linear and attention kernels at the edges of their tiles, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import sfo
from paper_2511_20340_amd import binding as sfb

from gpu_common import dev, engine_only, rel_err, to_np

pytestmark = pytest.mark.gpu


def shape_for(Hq, Hkv, hd):
    return synth.ModelShape("t", 1, Hq * hd, Hq, Hkv, hd, 256, 512, "f32")


# rows around the 16-row tiles (1 and 2 per workgroup), a column remainder of 8, K of one, one and a half, 16 and
# 32.5 chunks of 16 positions (1, 1, 4 and 8 waves), and the longest K split over all waves.  K products summed in
# fp32 in any order: relative error below K * 2^-24 <= 1.3e-4 of the absolute sums, in practice sqrt(K) * 2^-24.
@pytest.mark.parametrize("M", [1, 16, 17, 50])
@pytest.mark.parametrize("N,K", [(8, 8), (24, 24), (264, 256), (40, 520), (72, 2048)])
def test_linear_f32_tile_edges(M, N, K):
    g = synth.rng(31, M * 10007 + N * 31 + K)
    x = g.standard_normal((M, K), dtype=np.float32)
    w = g.standard_normal((N, K), dtype=np.float32) * 0.05
    bias = g.standard_normal(N, dtype=np.float32)
    res = g.standard_normal((M, N), dtype=np.float32)
    eng = engine_only(shape_for(2, 2, 64), 1, 64, 1)
    y = dev(res, "f32")
    eng.sf_op_linear(dev(x, "f32"), dev(w, "f32"), bias=dev(bias, "f32"), residual=y, y=y)
    assert rel_err(to_np(y), sfo.linear(x, w, bias) + res) < 1e-5
    few = eng.sf_op_linear(dev(x[:1], "f32"), dev(w, "f32"))
    whole = eng.sf_op_linear(dev(x, "f32"), dev(w, "f32"))
    torch.cuda.synchronize()
    assert torch.equal(few, whole[:1])          # a row does not depend on the rows batched with it


@pytest.mark.parametrize("M,F,K", [(1, 32, 8), (16, 96, 264), (33, 32, 1040)])
def test_linear_swiglu_f32_tile_edges(M, F, K):
    g = synth.rng(32, M + F + K)
    x = g.standard_normal((M, K), dtype=np.float32)
    w = g.standard_normal((2 * F, K), dtype=np.float32) * (2.0 / np.sqrt(K))
    eng = engine_only(shape_for(2, 2, 64), 1, 64, 1)
    act = eng.sf_op_linear_swiglu(dev(x, "f32"), dev(w, "f32"))
    assert rel_err(to_np(act), sfo.silu_mul(sfo.linear(x, w[:F]), sfo.linear(x, w[F:]))) < 1e-5


@pytest.mark.parametrize("mode", [sfb.SF_MASK_CAUSAL, sfb.SF_MASK_BIDIR])
@pytest.mark.parametrize("Hq,Hkv,hd,nq", [(4, 4, 8, 1), (8, 2, 24, 3), (2, 1, 256, 8), (4, 4, 64, 32)])
def test_attention_f32_head_sizes(mode, Hq, Hkv, hd, nq):
    # lengths: empty prefix, one key, around one and two chunks of 512 keys
    lens = np.array([0, 1, 511, 513, 1100], np.int32)
    cap = 1152
    q, kc, vc = synth.random_qkv(33, len(lens), nq, Hq, Hkv, hd, cap, "f32")
    ref = sfo.attention(q, kc, vc, lens, mode)
    for b in range(len(lens)):                  # nothing past the block may be read
        kc[b, :, lens[b] + nq:] = np.nan
        vc[b, :, lens[b] + nq:] = np.nan
    eng = engine_only(shape_for(Hq, Hkv, hd), len(lens), cap, max(nq - 1, 1))
    eng.sf_kv_import(kc, "dk"); eng.sf_kv_import(vc, "dv")
    out = eng.sf_op_attention(dev(q, "f32"), eng.dk, eng.dv, torch.from_numpy(lens).cuda(), nq, mode)
    assert rel_err(to_np(out), ref) < 1e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("first", [512, 700])
def test_attention_chunk_without_a_finite_score(dtype, first):
    """Keys whose scores are all -inf weigh nothing, also where they fill the first chunk of keys whole."""
    B, Hq, Hkv, hd, nq, cap = 2, 4, 2, 64, 3, 1152
    lens = np.array([1100, 800], np.int32)
    q, kc, vc = synth.random_qkv(37, B, nq, Hq, Hkv, hd, cap, dtype)
    q = np.abs(q) + 0.25
    ref = sfo.attention(synth.to_bf16_values(q), np.concatenate([kc[:, :, first:], kc[:, :, :first]], 2),
                        np.concatenate([vc[:, :, first:], vc[:, :, :first]], 2), lens - first, sfb.SF_MASK_CAUSAL)
    kc[:, :, :first] = -np.inf
    eng = engine_only(synth.ModelShape("t", 1, Hq * hd, Hq, Hkv, hd, 256, 512, dtype), B, cap, nq - 1)
    eng.sf_kv_import(kc, "dk"); eng.sf_kv_import(vc, "dv")
    out = to_np(eng.sf_op_attention(dev(synth.to_bf16_values(q), dtype), eng.dk, eng.dv, torch.from_numpy(lens).cuda(), nq,
                                    sfb.SF_MASK_CAUSAL))
    assert rel_err(out, ref) < (1e-5 if dtype == "f32" else 2e-2)      # the tolerances of the other attention tests


# K: one chunk and a half, 32.5 chunks over 8 waves, 65 over 16, 130 over 16 (shares that end off the four chunks in flight)
@pytest.mark.parametrize("M", [1, 17])
@pytest.mark.parametrize("K", [24, 520, 1040, 2080])
def test_linear_f32_infinite_weight_stays_in_its_column(M, K):
    g = synth.rng(38, K)
    x = np.abs(g.standard_normal((M, K), dtype=np.float32)) + 0.5
    w = g.standard_normal((40, K), dtype=np.float32)
    at = {5 * i: k for i, k in enumerate((0, K // 2, K - 1, K - 9, K // 4 + 3, K // 8, K // 16))}
    for n, k in at.items():
        w[n, k] = np.inf
    y = to_np(engine_only(shape_for(2, 2, 64), 1, 64, 1).sf_op_linear(dev(x, "f32"), dev(w, "f32")))
    cols = np.array(sorted(at))
    assert np.all(y[:, cols] == np.inf) and np.all(np.isfinite(np.delete(y, cols, 1)))
