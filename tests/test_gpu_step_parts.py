"""The decode step run as verify, one-workgroup-per-unit select and draft (short
contexts that do not take the one-kernel step) equals the separate calls, and
the one-launch greedy acceptance equals the oracle in every replay of a graph."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_27735_amd import binding as B

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU visible", allow_module_level=True)


@pytest.mark.parametrize("batch,hq,hkv,ctx,budget", [(1, 8, 2, 4096, 256), (2, 16, 4, 1500, 100), (1, 4, 4, 40, 64)])
def test_step_equals_the_separate_calls(batch, hq, hkv, ctx, budget):
    g = torch.Generator(device="cuda")
    g.manual_seed(ctx)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    q, qd = rnd(batch, 5, hq, 128), rnd(batch, hq, 128)
    k, v = rnd(batch, hkv, ctx + 3, 128), rnd(batch, hkv, ctx + 3, 128)
    lens, ql = [ctx - 7 * b for b in range(batch)], [5] * batch
    p = B.make_params(128 ** -0.5, budget=budget, out_fp32=True)
    assert not B.decode_step_plan(B.verify_shape(q, k), p, lens, ql)
    out, scores, idx, n_idx, dout = B.decode_step(q, k, v, qd, lens, ql, p)
    out_s, scores_s = B.verify_attn(q, k, v, lens, ql, p)
    idx_s, n_s = B.select_topb(scores_s, lens, p)
    n = [B.index_count(t, p.k_sink, p.k_recent, p.budget) for t in lens]
    dout_s = B.draft_attn(qd, k, v, idx_s, n, p)
    torch.cuda.synchronize()
    assert B.exchange_status() == 0
    assert torch.equal(out, out_s) and torch.equal(n_idx, n_s) and n_s.tolist() == n
    for b in range(batch):
        assert torch.equal(scores[b, :, :lens[b]], scores_s[b, :, :lens[b]])
        assert torch.equal(idx[b, :, :n[b]], idx_s[b, :, :n[b]])
    assert torch.equal(dout, dout_s)   # the same kernels in the same order


# (batch, query heads, KV heads, context, budget, positions, selected by a workgroup per unit?)
@pytest.mark.parametrize("batch,hq,hkv,ctx,budget,ql,unit", [
    (1, 4, 2, 16384, 512, 2, True), (1, 4, 2, 16385, 512, 2, False),    # the longest context
    (3, 16, 16, 4096, 1365, 1, True), (3, 16, 16, 4096, 1366, 1, False),    # 256 entries per CU
    (3, 8, 8, 4096, 4096, 1, True),                                      # and fewer partitions than half the CUs
    (2, 8, 8, 1000, 300, 1, True), (2, 8, 8, 1000, 1000, 1, False)])     # one partition, all selected
def test_the_steps_select_on_both_sides_of_its_lines(batch, hq, hkv, ctx, budget, ql, unit):
    """The step gives the bits of verify, select and draft, or of verify and
    select_draft, whichever its rule names."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the cases lie at the lines of 256 CUs")
    g = torch.Generator(device="cuda")
    g.manual_seed(ctx + budget)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    q, qd, k, v = (rnd(batch, ql, hq, 128), rnd(batch, hq, 128), rnd(batch, hkv, ctx, 128), rnd(batch, hkv, ctx, 128))
    lens, qls = [ctx] * batch, [ql] * batch
    p = B.make_params(128 ** -0.5, budget=budget, out_fp32=True, per_head=hq == hkv)   # (not the one-kernel step)
    if hq != hkv:
        assert not B.decode_step_plan(B.verify_shape(q, k), p, lens, qls)
    out, scores, idx, n_idx, dout = B.decode_step(q, k, v, qd, lens, qls, p)
    idx_u, n_u = B.select_topb(scores, lens, p, n_q_heads=hq)
    n = [B.index_count(t, p.k_sink, p.k_recent, p.budget) for t in lens]
    dout_u = B.draft_attn(qd, k, v, idx_u, n, p)
    idx_x, n_x, dout_x = B.select_draft(scores, lens, p, qd, k, v)
    torch.cuda.synchronize()
    assert B.exchange_status() == 0
    assert torch.equal(idx, idx_u) and torch.equal(idx, idx_x)
    assert torch.equal(dout, dout_u if unit else dout_x)
    assert ctx == 1000 or not torch.equal(dout_u, dout_x)   # (the two merge their partial results differently)


def test_a_step_that_drafts_over_most_rows_verifies_as_verify_attn():
    """A small step whose draft reads half of the cache again or more loads K and
    V without the streaming hint: the same bits as verify_attn's."""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    lens, qls = [4096, 4000, 3999, 4095, 3001], [2, 1, 2, 2, 1]
    q, qd, k, v = rnd(5, 2, 16, 128), rnd(5, 16, 128), rnd(5, 8, 4096, 128), rnd(5, 8, 4096, 128)
    p = B.make_params(128 ** -0.5, budget=4096, out_fp32=True)
    assert B.verify_plan(B.verify_shape(q, k), p, lens, qls)[0] == B.VERIFY_ONE_SWEEP_PERSISTENT
    out, scores, _, _, dout = B.decode_step(q, k, v, qd, lens, qls, p)
    out_v, scores_v = B.verify_attn(q, k, v, lens, qls, p)
    dout_x = B.select_draft(scores_v, lens, p, qd, k, v)[2]
    torch.cuda.synchronize()
    assert B.exchange_status() == 0
    assert torch.equal(out, out_v) and torch.equal(scores, scores_v) and torch.equal(dout, dout_x)


@pytest.mark.parametrize("vocab,k", [(17, 1), (8192, 3), (8193, 6), (128256, 5)])
def test_greedy_acceptance_in_a_graph(vocab, k):
    batch = 3
    rng = np.random.default_rng(vocab)
    stride = (vocab + 7) // 8 * 8   # (rows are 16-byte aligned)
    logits = torch.empty((batch, k + 1, stride), dtype=torch.float32, device="cuda")
    draft = torch.empty((batch, k), dtype=torch.int32, device="cuda")
    k_len = [k, 0, max(k - 1, 0)]
    cap = torch.cuda.Stream()
    logits.zero_(), draft.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(cap):
        B.greedy_accept(logits, draft, k_len, vocab=vocab)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        na, nxt = B.greedy_accept(logits, draft, k_len, vocab=vocab)
    for r in range(4):
        x = rng.standard_normal((batch, k + 1, stride)).astype(np.float32)
        d = x[:, :k, :vocab].argmax(-1).astype(np.int32)
        d[0, r % k] = (d[0, r % k] + r) % vocab    # a refusal, but in the first replay
        logits.copy_(torch.from_numpy(x))
        draft.copy_(torch.from_numpy(d))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        na_e, nxt_e = B.greedy_accept(logits, draft, k_len, vocab=vocab)
        torch.cuda.synchronize()
        ref = oracle.greedy_accept(x, d, np.asarray(k_len, np.int32), vocab=vocab)
        for got in ((na, nxt), (na_e, nxt_e)):
            assert np.array_equal(got[0].cpu().numpy(), ref[0]) and np.array_equal(got[1].cpu().numpy(), ref[1]), r
    assert B.exchange_status() == 0
