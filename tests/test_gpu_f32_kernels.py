"""fp32 mode: the linear and attention kernels at the edges of their tiles, against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import sfo
from paper_2511_20340_amd import binding as sfb
from paper_2511_20340_amd.engine import Engine

from gpu_common import dev, engine_only, rel_err, to_np

pytestmark = pytest.mark.gpu


def shape_for(Hq, Hkv, hd):
    return synth.ModelShape("t", 1, Hq * hd, Hq, Hkv, hd, 256, 512, "f32")


# rows around the 16-row tiles (1 and 2 per workgroup), a column remainder of 8, K of half a chunk of 16 positions, one and a
# half, 16 and 32.5 (1, 1, 8 and 16 waves), and a longer K over 16 waves.  K products summed in
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


# the kernel for many rows against the small one, which takes up to 63 of the same rows: tile edges in rows (128) and columns
# (64; 32 features with the gate), a remainder of 8 columns, K of half a chunk behind 5 (2 shares) and of 16 uneven shares
@pytest.mark.parametrize("M,N,K", [(64, 20488, 88), (1300, 1000, 1000), (4100, 320, 520), (129, 8200, 24)])
def test_linear_f32_many_rows_give_the_bits_of_few(M, N, K):
    assert M >= 64 and -(-N // 16) * -(-M // 32) >= 2560      # the rule's line
    g = torch.Generator(device="cuda").manual_seed(M)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x, w, bias, res = rand(M, K), rand(N, K) * 0.05, rand(N), rand(M, N)
    w[3, K - 1] = torch.inf
    x[:, K - 1] = x[:, K - 1].abs() + 0.5
    eng = engine_only(shape_for(2, 2, 64), 1, 64, 1)
    y = res.clone()
    eng.sf_op_linear(x, w, bias=bias, residual=y, y=y)
    Fw = w[8:8 + (N - 8) // 64 * 64]
    act = eng.sf_op_linear_swiglu(x, Fw)
    exact = x.double() @ w.double().T + bias.double() + res.double()
    finite = [n for n in range(N) if n != 3]
    assert bool((y[:, 3] == torch.inf).all())
    assert rel_err(to_np(y[:, finite]), exact[:, finite].cpu().numpy()) < 1e-5
    for first in sorted({0, 63, M // 2, max(0, M - 40)}):
        few = slice(first, min(first + 40, M))
        r = res[few].clone()
        eng.sf_op_linear(x[few].contiguous(), w, bias=bias, residual=r, y=r)
        assert torch.equal(r, y[few])
        assert torch.equal(eng.sf_op_linear_swiglu(x[few].contiguous(), Fw), act[few])


def test_step_f32_many_rows_give_the_bits_of_few():
    """A whole fp32 draft and verify step of 512 sequences (norm, gate, residual, hooked copies through the kernel for many
    rows) against the same sequences eight at a time."""
    shape, B, k, cap = synth.ModelShape("t", 2, 512, 4, 4, 128, 1024, 1024, "f32"), 512, 3, 64
    tw, dw = synth.target_weights(shape, 3), synth.draft_weights(shape, k, 3)
    g = synth.rng(39, 0)
    toks = g.integers(0, shape.vocab, (B, k + 1)).astype(np.int32)
    hooks = torch.from_numpy(g.standard_normal((B, k + 1, 4, 512), dtype=np.float32)).cuda()

    def step(rows):
        eng = Engine(shape.cfg(), len(rows), cap, k)
        eng.bind(tw, dw)
        eng.set_state(kv_len=np.full(len(rows), 2, np.int32), pending=toks[rows, 0], n_new=np.full(len(rows), 2, np.int32))
        eng.hooks.copy_(hooks[rows])
        dl = torch.empty(len(rows), k, shape.vocab, device="cuda")
        eng.sf_draft_step(k, logits_out=dl)
        logits, _ = eng.sf_verify_step(k, torch.from_numpy(toks[rows, 1:].copy()).cuda())
        torch.cuda.synchronize()
        return dl, logits.clone(), eng.hooks.clone()
    whole = step(np.arange(B))
    for first in (0, 256, B - 8):
        rows = np.arange(first, first + 8)
        for got, want in zip(whole, step(rows)):
            assert torch.equal(got[rows], want)
