"""Prefill in blocks longer than the decoding block runs every block over the prompts that have started (rows ordered by
length, caches in place).  It has to leave what running all prompts in every block leaves, bit for bit: caches with their
rows behind the prompts, lengths, choices, newest hooked states."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth

from paper_2511_20340_amd import binding as sfb
from paper_2511_20340_amd import engine as E

from gpu_common import linear_choice

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


# Where a part of the batch, planned for by itself, would sum in another order: half of 64 sequences in blocks of 16 split the
# K of the down projection and of the draft's 4d -> d projection, the whole does not; the 256 attention workgroups of the whole
# batch keep 21 key tiles in one chunk each, the 128 of half of it would cut them after 16 (512 keys).
WIDE = synth.ModelShape("t", 2, 1024, 8, 1, 64, 4096, 1032, "bf16")
HALF, ALL, BLOCK = 32, 64, 16


def test_bits_of_the_whole_batch_where_its_plan_matters():
    d, F = WIDE.d_model, WIDE.d_ffn
    for N, K in ((d, F), (d, 4 * d)):
        assert linear_choice(HALF * BLOCK, N, K)[2] == 4 and linear_choice(ALL * BLOCK, N, K)[2] == 1
    assert (8 * BLOCK + 31) // 32 * HALF == 128                  # attention workgroups per key chunk
    k, cap = 4, 704
    lens = [(600 + 13 * i) % 60 + 600 for i in range(HALF)] + [5 + i for i in range(ALL - HALF)]
    lens = [lens[(i * 27) % ALL] for i in range(ALL)]             # long and short ones mixed
    tw, dw = synth.target_weights(WIDE, 17, 0.05), synth.draft_weights(WIDE, k, 17, 0.05)
    eng, ref = (E.Engine(WIDE.cfg(), ALL, cap, k) for _ in range(2))
    eng.bind(tw, dw)
    ref.bind_shared(eng, with_draft=True)
    prompts = synth.prompts(lens, WIDE.vocab, 19)
    first = eng.prefill(prompts, block=BLOCK)
    helper = E.Engine(ref.cfg, ALL, cap, BLOCK - 1, share_caches=ref)
    helper.bind_shared(ref, with_draft=True)
    want = E._prefill_blocks(helper, prompts, BLOCK, k)
    torch.cuda.synchronize()
    assert torch.equal(first, want) and eng.kv_len.tolist() == lens
    for name in ("tk", "tv", "dk", "dv"):
        a, b = getattr(eng, name), getattr(ref, name)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name
    rows = helper.hooks[torch.arange(ALL), (helper.n_new.long() - 1).cpu()]
    assert torch.equal(eng.hooks[:, 0], rows)


@pytest.mark.parametrize("n,k_draft", [(HALF, 2), (HALF, 4), (24, 1), (1, 4)])
def test_last_block_over_a_part_of_the_batch(n, k_draft):
    """sf_prefill_step(last) over the first n rows leaves those sequences, in their cache slots, what the three steps over the
    whole batch leave them: the slots' layers are planned for the whole batch's rows too."""
    d, rows = WIDE.d_model, {1: (24, 64, 1024), 2: (64, 128, 1024), 4: (128, 256, 1024)}[k_draft]
    qkv = ((WIDE.n_q_heads + 2) * WIDE.head_dim, d)
    if n == HALF:      # the slots' QKV: split for half of the batch (k_draft 2: for all of it too), not for whole blocks
        assert [linear_choice(r, *qkv)[2] for r in rows] == {2: [2, 2, 1], 4: [2, 1, 1]}[k_draft]
    k, cap = BLOCK - 1, 64
    tw, dw = synth.target_weights(WIDE, 17, 0.05), synth.draft_weights(WIDE, k_draft, 17, 0.05)
    eng, ref = (E.Engine(WIDE.cfg(), ALL, cap, k) for _ in range(2))
    eng.bind(tw, dw)
    ref.bind_shared(eng, with_draft=True)
    g = synth.rng(71, n)
    tokens = torch.from_numpy(g.integers(0, WIDE.vocab, (2, ALL, BLOCK)).astype(np.int32)).cuda()
    size = torch.from_numpy(g.integers(1, BLOCK + 1, (2, ALL)).astype(np.int32)).cuda()
    slots = torch.from_numpy(g.permutation(ALL).astype(np.int32)).cuda()
    i32 = dict(dtype=torch.int32, device="cuda")
    ids, acc, out = torch.zeros(ALL, BLOCK, **i32), torch.empty(ALL, **i32), torch.empty(ALL, BLOCK, **i32)
    drafted = torch.full((ALL, k_draft), -7, **i32)
    ptr = lambda t: C.c_void_p(t.data_ptr())
    for e in (eng, ref):
        e.set_state(kv_len=np.zeros(ALL, np.int32), n_new=np.zeros(ALL, np.int32))
    for block in range(2):
        rest = tokens[block, :, 1:].contiguous()
        for e in (eng, ref):
            e.pending.copy_(tokens[block, :, 0])
        sfb.check(eng.lib.sf_prefill_step(eng.ctx, C.byref(eng.st), k, ptr(rest), ptr(size[block]), n, ptr(slots), BLOCK * block,
                                          BLOCK * (block + 1), k_draft, block, ptr(ids), ptr(acc), ptr(out), ptr(drafted),
                                          C.c_void_p(torch.cuda.current_stream().cuda_stream)), "sf_prefill_step", eng.ctx)
        ref.len_upper = BLOCK * block
        _, want_ids = ref.sf_verify_step(k, rest, logits=False)
        want_acc, want_out = ref.sf_accept_commit(k, rest, want_ids, force_len=size[block])
        ref.len_upper = BLOCK * (block + 1)
        want_draft = ref.sf_draft_step(k_draft)
    torch.cuda.synchronize()
    assert torch.equal(ids[:n], want_ids[:n]) and torch.equal(acc[:n], want_acc[:n]) and torch.equal(out[:n], want_out[:n])
    assert torch.equal(drafted[:n], want_draft[:n]) and not (drafted[n:] + 7).any()
    assert torch.equal(eng.kv_len[:n], ref.kv_len[:n]) and not eng.kv_len[n:].any()
    for j in range(n):             # committed rows of hooks; what lies behind them is scratch
        assert torch.equal(eng.hooks[j, :int(size[1, j])], ref.hooks[j, :int(size[1, j])])
    to = slots[:n].long()
    for name, layers in (("tk", 2), ("tv", 2), ("dk", 1), ("dv", 1)):
        for l in range(layers):
            a, b = eng.sf_kv_export(name, l), ref.sf_kv_export(name, l)
            assert torch.equal(a[to], b[:n]), (name, l)
            a[to] = 0
            assert not a.any(), name                      # nobody else's slot was written
