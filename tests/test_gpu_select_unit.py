"""The one-workgroup-per-unit select (calls of more than 256 partitions, contexts
of at most 65536 positions) against the oracle, index by index, at the edges of
its runs (8, 16, 32 scores per thread), rounds (32768) and candidate list."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
from paper_2607_27735_amd import binding as B

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU visible", allow_module_level=True)

# name: (context lengths, KV heads, k_sink, k_recent, budget); sequences are
# repeated until the call has more than 256 partitions
CASES = {
    "run8": ([8192, 8191, 33, 1, 5000, 37], 8, 4, 32, 100),
    "run16": ([8193, 16384, 8192 + 36, 40], 8, 4, 32, 1024),
    "run32": ([16385, 32768, 3, 20011], 8, 0, 0, 4096),
    "two-rounds": ([32769, 65536, 32768 + 36, 32768 + 37, 100], 4, 4, 32, 4096),
    # 30 units, enough for a workgroup per unit up to 65536 positions; 29 (and the 20 above) take
    # three kernels there
    "two-rounds-30": ([32769, 65536, 32768 + 36, 32768 + 37, 100], 6, 4, 32, 4096),
    "three-kernels-29": ([65536], 29, 4, 32, 4096),
}


def _scores(rng, kind, n, t):
    if kind == "log-normal":
        s = np.exp(1.2 * rng.standard_normal((n, t))) / t
    elif kind == "ties":       # 60 values, so that ties are cut in position order
        s = np.floor(rng.random((n, t)) * 60) / 64
    elif kind == "one-value":  # every position is a candidate and a tie
        s = np.full((n, t), 0.25)
    else:                      # most of them zero, of either sign, some huge
        s = np.where(rng.random((n, t)) < 0.95, 0.0, rng.random((n, t)) * 3e38)
        s[:, ::2] *= np.where(s[:, ::2] == 0.0, -1.0, 1.0)
    return s.astype(np.float32)


@pytest.mark.parametrize("kind", ["log-normal", "ties", "one-value", "zeros"])
@pytest.mark.parametrize("name", list(CASES))
def test_unit_select_matches_oracle(name, kind):
    base, hkv, k_sink, k_recent, budget = CASES[name]
    max_ctx = max(base) + 3
    params = B.make_params(0.1, k_sink=k_sink, k_recent=k_recent, budget=budget)
    ctx = list(base)
    while B.select_plan(B.Shape(len(ctx), hkv, hkv, 128, max_ctx, 1), params, ctx)[0]:
        ctx.append(base[len(ctx) % len(base)])
    print(f"[select] {name} {kind} ctx={ctx}", flush=True)
    rng = np.random.default_rng(len(ctx))
    s = _scores(rng, kind, len(ctx) * hkv, max_ctx).reshape(len(ctx), hkv, max_ctx)
    scores = torch.from_numpy(s).cuda()
    idx = torch.full((len(ctx), hkv, budget), -7, dtype=torch.int32, device="cuda")
    idx, n_idx = B.select_topb(scores, ctx, params, idx=idx)
    torch.cuda.synchronize()
    w = SimpleNamespace(batch=len(ctx), n_kv_heads=hkv)
    ref, n_ref = oracle.select(w, s, ctx_len=np.asarray(ctx, np.int32), k_sink=k_sink, k_recent=k_recent, budget=budget)
    got = idx.cpu().numpy()
    assert np.array_equal(n_idx.cpu().numpy(), n_ref)
    for b in range(len(ctx)):
        assert np.array_equal(got[b, :, :n_ref[b]], ref[b, :, :n_ref[b]]), f"sequence {b} of {ctx[b]}"
        assert np.all(got[b, :, n_ref[b]:] == -7)
