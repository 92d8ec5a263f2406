"""Prefill in blocks longer than the decoding block runs every block over the prompts that have started (rows ordered by
length, caches in place).  It has to leave what running all prompts in every block leaves, bit for bit: caches with their
rows behind the prompts, lengths, choices, newest hooked states."""
import numpy as np
import pytest
import torch

import synth

from paper_2511_20340_amd import binding as sfb
from paper_2511_20340_amd import engine as E

pytestmark = pytest.mark.gpu

SHAPES = {"bf16": synth.ModelShape("t", 3, 256, 8, 2, 64, 512, 1032, "bf16"),
          "f32": synth.ModelShape("t", 3, 256, 4, 4, 64, 512, 1024, "f32")}


def pair(dtype, B, cap, k, draft=True):
    m = SHAPES[dtype]
    tw, dw = synth.target_weights(m, 7, 0.05), synth.draft_weights(m, k, 7, 0.05) if draft else None
    engines = [E.Engine(m.cfg(), B, cap, k) for _ in range(2)]
    for e in engines:
        e.bind(tw, dw)
    return m, engines


# lengths: one token, one short of, at and above a block, several blocks, equal ones, the longest not first
@pytest.mark.parametrize("dtype", SHAPES)
@pytest.mark.parametrize("block,lens", [(16, [1, 15, 16, 17, 40, 40, 3, 64]), (8, [5, 30, 8, 8, 9]), (16, [20]), (16, [7, 7])])
def test_bits_of_all_prompts_in_every_block(dtype, block, lens):
    B, k, cap = len(lens), 4, 96
    m, (eng, ref) = pair(dtype, B, cap, k)
    prompts = synth.prompts(lens, m.vocab, 11)
    first = eng.prefill(prompts, block=block)
    helper = E.Engine(ref.cfg, B, cap, block - 1, share_caches=ref)
    helper.bind_shared(ref, with_draft=True)
    want = E._prefill_blocks(helper, prompts, block, k)
    torch.cuda.synchronize()
    assert torch.equal(first, want) and torch.equal(eng.pending, want)
    assert eng.kv_len.tolist() == lens and torch.equal(helper.kv_len, eng.kv_len) and eng.len_upper == max(lens)
    for name in ("tk", "tv", "dk", "dv"):
        a, b = getattr(eng, name), getattr(ref, name)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name
    rows = helper.hooks[torch.arange(B), (helper.n_new.long() - 1).cpu()]
    assert torch.equal(eng.hooks[:, 0], rows) and not eng.hooks[:, 1:].any() and eng.n_new.tolist() == [1] * B


def test_without_a_draft_and_with_an_empty_prompt():
    m, (eng, ref) = pair("bf16", 3, 96, 4, draft=False)
    prompts = synth.prompts([33, 2, 50], m.vocab, 12)
    eng.prefill(prompts, block=16)
    assert eng.kv_len.tolist() == [33, 2, 50] and not eng.dk.any()
    ref.prefill([prompts[0], prompts[1][:0], prompts[2]], block=16)   # all prompts in every block
    assert ref.kv_len.tolist() == [33, 0, 50] and ref.n_new.tolist() == [1, 0, 1]
    assert torch.equal(ref.pending[[0, 2]], eng.pending[[0, 2]])


def test_refuses_what_does_not_fit():
    m, (eng, _) = pair("bf16", 2, 64, 4)
    with pytest.raises(sfb.SfError) as err:
        eng.prefill(synth.prompts([20, 62], m.vocab, 13), block=16)      # the prompt fits, its draft slots do not
    assert err.value.status == sfb.SF_ECAPACITY
    with pytest.raises(sfb.SfError) as err:
        eng.prefill(synth.prompts([20, 90], m.vocab, 13), block=16)
    assert err.value.status == sfb.SF_ECAPACITY
