"""Vocabularies that are no multiple of 8: the LM head's logits end within the epilogue's groups of 8 columns."""
import numpy as np
import pytest
import torch

import synth
from paper_2511_20340_amd.engine import Engine

pytestmark = pytest.mark.gpu

CAP, K = 64, 4


def step(V, weights, B, d, tokens):
    """A draft and a verify step; logits land in the middle of buffers of a known value."""
    tw, dw = weights
    eng = Engine(synth.ModelShape("t", 1, d, 2, 2, 64, 128, V, "bf16").cfg(), B, CAP, K)
    eng.bind(dict(tw, embed=tw["embed"][:V], lm_head=tw["lm_head"][:V]), dw)
    eng.set_state(kv_len=np.full(B, 1, np.int32), pending=tokens[:, 0], n_new=np.ones(B, np.int32))
    out = []
    for rows in (K, K + 1):
        room = torch.full((64 + B * rows * V + 64,), 12345.0, device="cuda")
        logits = room[64:64 + B * rows * V].view(B, rows, V)
        if rows == K:
            ids = eng.sf_draft_step(K, logits_out=logits)
        else:
            _, ids = eng.sf_verify_step(K, torch.from_numpy(tokens[:, 1:].copy()).cuda(), logits_out=logits)
        torch.cuda.synchronize()
        assert bool((room[:64] == 12345.0).all()) and bool((room[-64:] == 12345.0).all())
        out.append((logits.clone(), ids.clone()))
    return out


# rows: ring tiles of 32 and 160 rows, block tiles (d a multiple of 64) around 330; vocabularies: within one group of 8, 5, 4
# and 1 columns past one, a float row that starts on 16 bytes (4) or does not (1, 5)
@pytest.mark.parametrize("d", [256, 264])
@pytest.mark.parametrize("B", [1, 9, 66])
@pytest.mark.parametrize("V", [5, 77, 516, 1025])
def test_odd_vocabulary(V, B, d):
    weights = synth.target_weights(synth.ModelShape("t", 1, d, 2, 2, 64, 128, 1032, "bf16"), 3, 0.1)
    draft = synth.draft_weights(synth.ModelShape("t", 1, d, 2, 2, 64, 128, 1032, "bf16"), K, 3, 0.1)
    tokens = synth.rng(5, V + B).integers(0, V, (B, K + 1)).astype(np.int32)
    want = step(1032, (weights, draft), B, d, tokens)        # the same head with more rows
    for (logits, ids), (ref, _) in zip(step(V, (weights, draft), B, d, tokens), want):
        assert torch.equal(logits, ref[:, :, :V])
        assert torch.equal(ids.long(), ref[:, :, :V].argmax(-1))
