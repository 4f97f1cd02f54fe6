"""GPU parity of the streaming one-sweep verify kernel (two workgroups per CU;
verify_stream.hip) at the edges of its tiles and chunks.

Both stash forms: 16-bit codes (reached with a small CU budget, so that small
shapes take several chunks per unit) and fp32 (contexts of more than 64 code
chunks per head).  Outputs and scores are held to the oracle bars; the fp32
form's scores, sums of fp32 probabilities, to 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import Dev, abs_v, check_outputs, check_score_mass, check_scores, dev_bf16
from paper_2607_27735_amd import binding as B
from paper_2607_27735_amd.workloads import bf16_bits_to_f32, f32_to_bf16_bits, generate

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU visible", allow_module_level=True)

NAN_BF16 = np.uint16(0x7FC0)


def _poison(w):
    for b in range(w.batch):
        w.k[b, :, w.ctx_len[b]:] = NAN_BF16
        w.v[b, :, w.ctx_len[b]:] = NAN_BF16
        w.q[b, w.q_len[b]:] = NAN_BF16
    return w


def _gen(seed, ctx, ql, hq, hkv, spare=3):
    return _poison(generate(seed, name="stream", batch=len(ctx), n_q_heads=hq, n_kv_heads=hkv,
                            ctx_len=ctx, q_len=ql, max_ctx=max(ctx) + spare, max_q=max(ql),
                            budget=64, heavy_hitters=0))


def _ramp(w, top):
    """Every key's logits rise along the context to about `top` (log2 units):
    the reference maxima move again and again."""
    for b in range(w.batch):
        T = int(w.ctx_len[b])
        for c in range(w.n_kv_heads):
            rows = bf16_bits_to_f32(w.q[b, :w.q_len[b], c * w.group:(c + 1) * w.group]).reshape(-1, 128)
            u = rows.mean(axis=0).astype(np.float64)
            u /= u @ u                      # one unit of the mean query's product
            k = bf16_bits_to_f32(w.k[b, c, :T]).astype(np.float64) * 0.2
            k += (np.arange(T)[:, None] / T) * (top / (w.sm_scale * 1.4427)) * u
            w.k[b, c, :T] = f32_to_bf16_bits(k.astype(np.float32))
    return w


def _shift(w, by):
    """Every logit moves by about `by` (log2 units): the queries of a sequence
    get a shared part, the keys the multiple of it that gives the shift."""
    rng = np.random.default_rng(7)
    for b in range(w.batch):
        a = rng.standard_normal(128)
        q = 0.25 * bf16_bits_to_f32(w.q[b]) + a
        k = bf16_bits_to_f32(w.k[b]) + a * (by / (w.sm_scale * 1.4427 * (a @ a)))
        w.q[b], w.k[b] = f32_to_bf16_bits(q.astype(np.float32)), f32_to_bf16_bits(k.astype(np.float32))
    return w


# name: (workload, CU budget or 0, 16-bit codes?)
CASES = {
    # one and two keys past a tile and a chunk; 12 rows; single-chunk units; T below a tile
    "codes-rows12": (lambda: _gen(801, [4097, 1057, 31, 2050], [3, 3, 1, 2], 8, 2), 5, True),
    # 17 and 31 rows (a second row tile begun and nearly full), group not a power of two
    "codes-group31": (lambda: _gen(802, [2500, 1601], [1, 1], 31, 1), 4, True),
    "codes-rows17": (lambda: _gen(803, [2500, 1], [17, 1], 1, 1), 4, True),
    # 33 rows, logits that rise by 120 octaves
    "codes-ramp33": (lambda: _ramp(_gen(804, [3000, 1500], [11, 5], 6, 2), 120.0), 6, True),
    # logits near -300 (log2 units); a last chunk of two keys, none of which the first row may see
    "codes-low": (lambda: _poison(_shift(_gen(812, [2050], [3], 8, 1), -300.0)), 5, True),
    # fp32: ragged long contexts, 40, 8 and 36 rows
    "fp32-rows40": (lambda: _gen(805, [44999, 300, 20001], [10, 2, 9], 16, 4), 0, False),
    # fp32, logits that rise by 120 octaves: stashed probabilities are rescaled
    "fp32-ramp40": (lambda: _ramp(_gen(806, [45056], [10], 16, 4), 120.0), 0, False),
    # fp32 in row blocks of 32 rows: 128, 72 (a partial last block) and 16 rows (one block); more
    # than eight chunks, not a multiple of eight
    "fp32-blocks128": (lambda: _gen(807, [4500, 1057, 517], [16, 9, 2], 16, 2), 0, False),
    # three blocks of four positions, the last of three; a sequence of one key
    "fp32-blocks88": (lambda: _gen(808, [1, 2000], [1, 11], 8, 1), 0, False),
    # a window of 16 positions: the first of three blocks has no rows in it
    "fp32-blocks-window": (lambda: _gen(810, [2000], [40], 2, 1), 0, False),
}


@pytest.fixture(autouse=True)
def _reset():
    torch.cuda.synchronize()
    B.exchange_status()
    yield
    B.set_cu_budget(0)


@pytest.mark.parametrize("per_head", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_stream_matches_oracle(name, per_head):
    make, budget, codes = CASES[name]
    w = make()
    print(f"[stream] {name} {w.describe()} per_head={per_head}", flush=True)
    d = Dev(w)
    B.set_cu_budget(budget)
    p = B.make_params(w.sm_scale, window=w.window, budget=w.budget, out_fp32=True, per_head=per_head)
    sch, chunk, items = B.verify_plan(B.verify_shape(d.q, d.k), p, w.ctx_len, w.q_len)
    assert sch == B.VERIFY_ONE_SWEEP_PERSISTENT, (sch, chunk, items)
    if name == "codes-low":
        assert w.ctx_len[0] % chunk == 2
    heads = w.n_q_heads if per_head else w.n_kv_heads
    out = torch.full(d.q.shape, -7.0, dtype=torch.float32, device="cuda")
    sc = torch.full((w.batch, heads, w.max_ctx), -1.0, dtype=torch.float32, device="cuda")
    B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, out=out, scores=sc)
    torch.cuda.synchronize()
    assert B.exchange_status() == 0
    o, s = out.double().cpu().numpy(), sc.double().cpu().numpy()
    o_ref, s_ref = oracle.verify(w)
    if per_head:
        s_ref = oracle.head_scores(w)
    mask = np.arange(w.max_q)[None, :, None] < w.q_len[:, None, None] * np.ones((1, 1, w.n_q_heads), bool)
    oabs, _ = oracle.verify(w, v=abs_v(w))
    check_outputs(o, o_ref, oabs, mask)
    assert np.all(o[~mask] == -7.0)
    tol = 1e-3 if codes else 4.3e-5 if "ramp" in name else 1e-5
    for b in range(w.batch):
        T = int(w.ctx_len[b])
        assert np.all(s[b, :, T:] == -1.0)
        # every key within 1e-3 (codes) or 1e-5 (fp32) of its score; logits near 2^7 log2 units
        # carry fp32 errors of a few ulps, 2^-16 each, so the ramp's probabilities one of
        # 4 * 2^-16 * ln 2 = 4.3e-5; keys below 2^-40 of the largest score may be flushed relative
        # to the reference maxima
        r, g = s_ref[b, :, :T], s[b, :, :T]
        big = r > r.max() * 2.0 ** -40
        assert np.abs(g - r)[big].max() == 0 or (np.abs(g - r)[big] / r[big]).max() <= tol
        assert np.all(g >= 0) and np.all(g[~big] <= r.max() * 2.0 ** -39)
    if not per_head:
        check_score_mass(s, w)
    if "ramp" not in name:
        check_scores(s, s_ref, w.ctx_len)


@pytest.mark.parametrize("name", ["codes-rows12", "fp32-rows40", "fp32-blocks128"])
def test_paged_and_bf16_outputs_give_the_dense_bits(name):
    """Over a shuffled page pool every form gives the dense call's bits, and its
    bf16 outputs are the fp32 ones, rounded."""
    from test_gpu_paged import paged
    make, budget, _ = CASES[name]
    w = make()
    d = Dev(w)
    B.set_cu_budget(budget)
    p, p16 = (B.make_params(w.sm_scale, window=w.window, budget=w.budget, out_fp32=f) for f in (True, False))
    assert B.verify_plan(B.verify_shape(d.q, d.k), p, w.ctx_len, w.q_len)[0] == B.VERIFY_ONE_SWEEP_PERSISTENT
    out, sc = B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p)
    out16, sc16 = B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p16)
    kp, vp, bt, _ = paged(w, 64, seed=17)
    kp, vp, bt = dev_bf16(kp), dev_bf16(vp), torch.from_numpy(bt).cuda()
    out_p, sc_p = B.verify_attn_paged(d.q, kp, vp, bt, w.max_ctx, w.ctx_len, w.q_len, p)
    out_p16, _ = B.verify_attn_paged(d.q, kp, vp, bt, w.max_ctx, w.ctx_len, w.q_len, p16)
    torch.cuda.synchronize()
    assert B.exchange_status() == 0
    assert torch.equal(out_p, out) and torch.equal(sc_p, sc) and torch.equal(sc16, sc)
    assert torch.equal(out16, out.to(torch.bfloat16)) and torch.equal(out_p16, out16)


def test_row_blocks_under_capture():
    """A captured call in row blocks: every replay, with eager calls between,
    equals the eager call on the same inputs."""
    w = _gen(809, [3000, 1057], [16, 9], 16, 2)
    d = Dev(w)
    p = B.make_params(w.sm_scale, window=w.window, budget=w.budget, out_fp32=True)
    assert B.verify_plan(B.verify_shape(d.q, d.k), p, w.ctx_len, w.q_len)[0] == B.VERIFY_ONE_SWEEP_PERSISTENT
    out = torch.empty(d.q.shape, dtype=torch.float32, device="cuda")
    sc = torch.zeros((w.batch, w.n_kv_heads, w.max_ctx), dtype=torch.float32, device="cuda")
    cap = torch.cuda.Stream()
    with torch.cuda.stream(cap):
        B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, out=out, scores=sc)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, out=out, scores=sc)
    base = d.q.clone()
    for r in range(4):
        d.q.copy_(base * (1.0 - 0.125 * r))
        out_e, sc_e = torch.empty_like(out), torch.zeros_like(sc)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, out=out_e, scores=sc_e)
        torch.cuda.synchronize()
        for b in range(w.batch):
            assert torch.equal(out[b, :w.q_len[b]], out_e[b, :w.q_len[b]]), f"replay {r}"
        assert torch.equal(sc, sc_e), f"replay {r}"
    assert B.exchange_status() == 0


@pytest.mark.parametrize("name", ["codes-rows12", "fp32-rows40", "fp32-blocks128"])
def test_a_nan_row_stays_in_its_row(name):
    """One verify row of one head is NaN (in fp32-rows40 of a unit of more than
    64 chunks, whose row sums several waves merge): the other rows and the other
    KV heads' scores keep their values, no wait gives up, and a captured call
    whose inputs are finite again is right again."""
    make, budget, _ = CASES[name]
    w = make()
    d = Dev(w)
    B.set_cu_budget(budget)
    p = B.make_params(w.sm_scale, window=w.window, budget=w.budget, out_fp32=True)
    sch, chunk, items = B.verify_plan(B.verify_shape(d.q, d.k), p, w.ctx_len, w.q_len)
    assert sch == B.VERIFY_ONE_SWEEP_PERSISTENT
    print(f"[stream] NaN row, {name}: chunks of {chunk}, {items} items", flush=True)
    if name == "fp32-rows40":
        assert w.ctx_len[0] > 64 * chunk
    out = torch.full(d.q.shape, -7.0, dtype=torch.float32, device="cuda")
    sc = torch.full((w.batch, w.n_kv_heads, w.max_ctx), -1.0, dtype=torch.float32, device="cuda")
    call = lambda: B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, out=out, scores=sc)
    call()
    torch.cuda.synchronize()
    good = out.clone(), sc.clone()
    row, head = (0, int(w.q_len[0]) - 1, w.group), 1   # the first query head of KV head 1
    cap = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        call()
    for run in (call, graph.replay):
        q = d.q.clone()
        d.q[row][:] = float("nan")
        out.fill_(-7.0)
        sc.fill_(-1.0)
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        assert B.exchange_status() == 0
        assert torch.isnan(out[row]).all()
        o, s = out.clone(), sc.clone()
        o[row] = good[0][row]
        s[0, head] = good[1][0, head]
        assert torch.equal(o, good[0]) and torch.equal(s, good[1])
        d.q.copy_(q)
        run()
        torch.cuda.synchronize()
        assert torch.equal(out, good[0]) and torch.equal(sc, good[1]) and B.exchange_status() == 0


def test_row_blocks_give_up_cleanly():
    """Row blocks whose waits all give up write neither outputs nor scores (the
    copies of the scores in the workspace hold other data), eager and captured;
    under capture they keep giving up until the workspace is cleared."""
    w = _gen(811, [3000, 1057], [16, 9], 16, 2)
    d = Dev(w)
    p = B.make_params(w.sm_scale, window=w.window, budget=w.budget, out_fp32=True)
    shape = B.verify_shape(d.q, d.k)
    assert B.verify_plan(shape, p, w.ctx_len, w.q_len)[0] == B.VERIFY_ONE_SWEEP_PERSISTENT
    ws = torch.full((B.verify_workspace_bytes(shape, p, w.ctx_len, w.q_len),), 0x3F, dtype=torch.uint8,
                    device="cuda")
    out = torch.full(d.q.shape, -7.0, dtype=torch.float32, device="cuda")
    sc = torch.full((w.batch, w.n_kv_heads, w.max_ctx), -1.0, dtype=torch.float32, device="cuda")
    call = lambda: B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, out=out, scores=sc, workspace=ws)

    def unwritten():
        torch.cuda.synchronize()
        return (B.exchange_status() == B.EXCHANGE_VERIFY and bool(torch.all(out == -7.0)) and
                bool(torch.all(sc == -1.0)))

    try:
        B.test_exchange_faults(64, True)
        call()
        assert unwritten()
        cap, bad, ok = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(bad, stream=cap):
            call()
        B.test_exchange_faults(0, False)
        with torch.cuda.graph(ok, stream=cap):
            call()
        bad.replay()
        assert unwritten()
        for _ in range(2):   # the clean graph finds the epochs marked
            ok.replay()
            assert unwritten()
    finally:
        B.test_exchange_faults(0, False)
    call()                   # an eager call uses no epochs
    torch.cuda.synchronize()
    good = out.clone(), sc.clone()
    out_ref, s_ref = oracle.verify(w)
    check_scores(sc.double().cpu().numpy(), s_ref, w.ctx_len)
    ws.fill_(0)
    for _ in range(2):
        out.fill_(-7.0)
        sc.fill_(-1.0)
        torch.cuda.synchronize()
        ok.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, good[0]) and torch.equal(sc, good[1]) and B.exchange_status() == 0


def test_a_smaller_workspace_takes_two_sweeps():
    """Row blocks need more workspace than two sweeps do, also than those of a
    longer context.  A call whose workspace holds the two sweeps only runs them,
    also as part of a decode step; with one byte less it is refused."""
    w = _gen(813, [3000, 1057], [16, 9], 16, 2)
    d = Dev(w)
    shape = B.verify_shape(d.q, d.k)
    p2, p = (B.make_params(w.sm_scale, window=w.window, budget=w.budget, out_fp32=True, verify_mode=m)
             for m in (B.VERIFY_TWO_SWEEP, B.VERIFY_AUTO))
    assert B.verify_plan(shape, p, w.ctx_len, w.q_len)[0] == B.VERIFY_ONE_SWEEP_PERSISTENT
    calls = {
        B.verify_workspace_bytes: lambda p, ws: B.verify_attn(d.q, d.k, d.v, w.ctx_len, w.q_len, p, workspace=ws),
        B.decode_step_workspace_bytes: lambda p, ws: B.decode_step(d.q, d.k, d.v, d.qd, w.ctx_len, w.q_len, p,
                                                                   workspace=ws),
    }
    for size, call in calls.items():
        small = size(shape, p2, w.ctx_len, w.q_len)
        assert size(shape, p, w.ctx_len, w.q_len) > small
        ref = call(p2, None)
        ws = torch.zeros(small, dtype=torch.uint8, device="cuda")
        got = call(p, ws)
        torch.cuda.synchronize()
        assert ws.any()    # the call ran in it
        assert all(torch.equal(a, b) for a, b in zip(ref, got))
        ws.zero_()
        call(p, ws[:-1])   # too small: the binding gives the call a workspace of its own
        torch.cuda.synchronize()
        assert not ws.any()


def test_static_scratch_takes_two_sweeps_where_row_blocks_need_more():
    """32 row blocks whose score copies exceed the library's 128 MiB: the entry
    point without a workspace runs two sweeps, which fit."""
    dev, g = torch.device("cuda:0"), torch.Generator(device="cuda:0")
    g.manual_seed(814)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device=dev).to(torch.bfloat16)
    q, k, v = rnd(8, 64, 32, 128), rnd(8, 2, 70000, 128), rnd(8, 2, 70000, 128)
    ctx, ql = [700, 333, 64, 512, 700, 129, 600, 301], [64, 7, 64, 33, 64, 64, 1, 64]
    p, p2 = (B.make_params(128 ** -0.5, budget=64, out_fp32=True, verify_mode=m)
             for m in (B.VERIFY_AUTO, B.VERIFY_TWO_SWEEP))
    shape = B.verify_shape(q, k)
    assert B.verify_plan(shape, p, ctx, ql)[0] == B.VERIFY_ONE_SWEEP_PERSISTENT
    assert B.verify_workspace_bytes(shape, p, ctx, ql) > (128 << 20) > B.verify_workspace_bytes(shape, p2, ctx, ql)
    ref = B.verify_attn(q, k, v, ctx, ql, p2)
    out, sc = torch.zeros_like(ref[0]), torch.zeros_like(ref[1])
    B.verify_attn_static(q, k, v, ctx, ql, p, out=out, scores=sc)
    torch.cuda.synchronize()
    assert torch.equal(out, ref[0]) and torch.equal(sc, ref[1])


def test_four_streams_at_once():
    """Streaming calls queued on four streams together, each with a workspace of
    its own (long groups of one block of 40 rows, two and four row blocks, more
    workgroups in each call than the device holds): every call gives the bits it
    gives alone and no wait gives up."""
    dev, g = torch.device("cuda:0"), torch.Generator(device="cuda:0")
    g.manual_seed(815)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device=dev).to(torch.bfloat16)
    p = B.make_params(128 ** -0.5, budget=64, out_fp32=True)
    calls = []
    # (query heads, KV heads, contexts, positions)
    for hq, hkv, ctx, n in [(16, 4, [60001, 44999], 10), (64, 8, [40011], 16), (32, 8, [40000], 16),
                            (64, 8, [9000, 8003], 16)]:
        q, k, v = rnd(len(ctx), n, hq, 128), rnd(len(ctx), hkv, max(ctx), 128), rnd(len(ctx), hkv, max(ctx), 128)
        ql, shape = [n] * len(ctx), B.verify_shape(q, k)
        sch, chunk, items = B.verify_plan(shape, p, ctx, ql)
        print(f"[stream] four streams: {hq}/{hkv} heads, {ctx} keys, {n} positions: {sch}, {chunk}, {items}", flush=True)
        assert sch == B.VERIFY_ONE_SWEEP_PERSISTENT and items > 512
        out = torch.zeros(q.shape, dtype=torch.float32, device=dev)
        sc = torch.zeros((len(ctx), hkv, max(ctx)), dtype=torch.float32, device=dev)
        ws = torch.empty(B.verify_workspace_bytes(shape, p, ctx, ql), dtype=torch.uint8, device=dev)
        st = torch.cuda.Stream()
        call = lambda a=(q, k, v, ctx, ql, p, out, sc, ws, st): B.verify_attn(*a)
        calls.append((call, out, sc))
    ref = []
    for call, out, sc in calls:
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        ref.append((out.clone(), sc.clone()))
    for _, out, sc in calls:
        out.zero_()
        sc.zero_()
    torch.cuda.synchronize()
    for _ in range(20):
        for call, _, _ in calls:
            call()
    torch.cuda.synchronize()
    assert B.exchange_status() == 0
    for (_, out, sc), (o, s) in zip(calls, ref):
        assert torch.equal(out, o) and torch.equal(sc, s)
