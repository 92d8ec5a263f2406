"""The merge of a split-KV attention's chunks, bit for bit: from the partial results that the chunks left in the workspace,
a row's sum and outputs are added chunk by chunk, each product and addition rounded once (fused multiply-add)."""
import numpy as np
import pytest
import torch

import synth
from paper_2511_20340_amd import binding as sfb

from gpu_common import engine_only

pytestmark = pytest.mark.gpu

CHUNK = 16 * 32      # keys


def fma(a, b, c):
    """a * b + c of float32 values, rounded once: the product is exact in float64."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


# The outputs are bf16, which hides most last-bit differences: half a million of them, so that some show.
# one chunk (nothing to merge), two, a few and a tail; forty: more than the 32 that one round of lanes holds
@pytest.mark.parametrize("Hq,Hkv,hd,nq,chunks", [(32, 8, 128, 20, 7), (16, 1, 64, 20, 40)])
def test_combine_adds_chunk_by_chunk_with_one_rounding(Hq, Hkv, hd, nq, chunks):
    cap, G = chunks * CHUNK, Hq // Hkv
    lens = np.array([100, 2 * CHUNK - nq] + [CHUNK * (1 + i % (chunks - 1)) + 90 * i for i in range(1, 8)] + [cap - nq] * 8, np.int32)
    B = len(lens)
    g = torch.Generator(device="cuda").manual_seed(71)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    eng = engine_only(synth.ModelShape("t", 1, Hq * hd, Hq, Hkv, hd, 256, 512, "bf16"), B, cap, nq - 1)
    eng.sf_kv_import(rand(B, Hkv, cap, hd), "dk"); eng.sf_kv_import(rand(B, Hkv, cap, hd), "dv")
    eng.sf_tune_attention(CHUNK // 32)
    out = eng.sf_op_attention(rand(B, nq, Hq, hd), eng.dk, eng.dv, torch.from_numpy(lens).cuda(), nq, sfb.SF_MASK_CAUSAL)
    torch.cuda.synchronize()

    n_rt, n_chunks = (G * nq + 31) // 32, chunks
    slots = eng.lib.sf_attention_workspace_bytes(eng.ctx, B, nq, int(lens.max())) // ((hd + 2) * 4)
    assert slots == B * Hkv * n_chunks * n_rt * 32
    ws = eng._keep_ws[(-eng._keep_ws.data_ptr()) % 256:]
    part = ws[:slots * (hd + 2) * 4].view(torch.float32)
    part_o = part[:slots * hd].view(B, Hkv, n_chunks, n_rt * 32, hd)
    part_ml = part[slots * hd:].view(B, Hkv, n_chunks, n_rt * 32, 2)
    for b in range(1, B):
        sc = -(-(int(lens[b]) + nq) // CHUNK)
        o_c = part_o[b, :, :sc, :G * nq].cpu().numpy()                    # [Hkv][sc][rows][hd]
        m, l_c = part_ml[b, :, :sc, :G * nq].unbind(-1)
        f = torch.exp2(m - m.amax(1, keepdim=True)).cpu().numpy()         # the device's own exponential
        l_c = l_c.cpu().numpy()
        l, o = np.zeros_like(f[:, 0]), np.zeros_like(o_c[:, 0])
        for c in range(sc):
            l = fma(l_c[:, c], f[:, c], l)
            o = fma(o_c[:, c], np.broadcast_to(f[:, c, :, None], o.shape), o)
        want = torch.from_numpy(o * (np.float32(1) / l)[..., None]).bfloat16()
        got = out[b].reshape(nq, Hkv, G, hd).permute(1, 0, 2, 3).reshape(Hkv, nq * G, hd).cpu()
        assert torch.equal(got, want), b
