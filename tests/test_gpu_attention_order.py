"""The order in which a step's attention workgroups start follows the sequences' lengths (descending, or what goes beyond one
workgroup per compute unit turned round); whatever it is, a sequence's results are the same bits as in a small batch that is
not ordered."""
import numpy as np
import pytest
import torch

import synth
from paper_2511_20340_amd.engine import Engine

pytestmark = pytest.mark.gpu

SHAPE = synth.ModelShape("t", 1, 512, 8, 8, 64, 256, 512, "bf16")
CAP, K = 160, 2


def step(rows, lens, caches, pending, draft, weights):
    """One verify step of the sequences `rows`; linear layers forced to one tile and split, so that only attention and
    its order can tell the batches apart."""
    B = len(rows)
    eng = Engine(SHAPE.cfg(), B, CAP, K)
    eng.bind(weights, None)
    for which, c in zip(("tk", "tv"), caches):
        eng.sf_kv_import(c[rows].contiguous(), which, 0)
    eng.set_state(kv_len=lens[rows], pending=pending[rows], n_new=np.ones(B, np.int32))
    eng.sf_tune_linear(2, 1)
    logits, _ = eng.sf_verify_step(K, torch.from_numpy(draft[rows]).cuda())
    torch.cuda.synchronize()
    return logits.clone(), eng.sf_kv_export("tk", 0).clone()


# 8 kv heads: 264, 384 and 512 workgroups (turned round from place 32 on: one, 16 and 32 sequences), 520 (descending)
@pytest.mark.parametrize("B", [33, 48, 64, 65])
def test_order_leaves_the_results(B):
    g = synth.rng(61, B)
    weights = synth.target_weights(SHAPE, 7)
    lens = g.integers(1, CAP - K - 1, B).astype(np.int32)
    lens[B // 2:] = np.sort(lens[B // 2:])               # ties and runs among them
    lens[1] = lens[0]
    gen = torch.Generator(device="cuda").manual_seed(B)
    caches = [torch.randn(B, 8, CAP, 64, generator=gen, device="cuda").bfloat16() for _ in range(2)]
    pending = g.integers(0, SHAPE.vocab, B).astype(np.int32)
    draft = g.integers(0, SHAPE.vocab, (B, K)).astype(np.int32)
    got_l, got_k = step(np.arange(B), lens, caches, pending, draft, weights)
    for first in range(0, B, 16):
        rows = np.arange(first, min(first + 16, B))      # 128 workgroups: no order
        want_l, want_k = step(rows, lens, caches, pending, draft, weights)
        assert torch.equal(got_l[rows], want_l) and torch.equal(got_k[rows], want_k)
