"""GPU parity of the decoding of short rows: every token scored, no partials, one launch.

Rows of at most 64 tokens, and of at most 256 in batches from 512, take a wave each; others a
workgroup each, up to 640 tokens, or 1024 in launches of at most 2^20 logits.  Both sides of
each of these lines and of a lane's four steps, with ties, NaNs, signed zeros and infinities,
shards, odd strides, both dtypes, seedings and windows; tokens equal the oracle's, values bit
for bit (NaN as NaN), the workspace untouched.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_argmax import assert_argmax_equal, hard_rows
from test_gpu_parity import WIDE, _to_device, env, say  # noqa: F401
from test_gpu_sample import seeds_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seeding,width", [("context", 3), ("self_salt", 1), ("self_salt", 4), ("self_salt", 7)])
@pytest.mark.parametrize("B,V", [(1, 1), (5, 63), (7, 64), (6, 65), (513, 65), (511, 256), (514, 256), (515, 257),
                                 (4, 640), (1639, 640), (1638, 641), (1024, 1024), (1025, 1024), (3, 1025)])
def test_short_rows(env, dtype, seeding, width, B, V):
    torch, sbw, dev = env
    rng = np.random.default_rng(B * 3 + V + width)
    x = hard_rows(rng, B, V, dtype)
    x[-1, V // 2:] = x[-1, V // 2]                    # ties across lanes and waves
    ctx = workloads.context_tokens(B, width, max(V, 2), rng)
    seeds = seeds_for(rng, B)
    base = np.zeros((B, V + 3), dtype=x.dtype)
    base[:, 1:V + 1] = x
    t = _to_device(torch, dev, base)[:, 1:V + 1]
    c = torch.from_numpy(np.ascontiguousarray(ctx, dtype=np.int32)).to(dev)
    s = torch.from_numpy(seeds.view(np.int64)).to(dev)
    ws = torch.full((sbw.argmax_workspace_size(B, V),), -5, dtype=torch.int64, device=dev)
    short = V <= 640 or V <= 1024 and B * V <= 1 << 20
    for gamma, delta in ((0.25, 2.0), (0.0, 1.0)):
        say(f"short rows {dtype} {seeding} h={width} B={B} V={V} gamma={gamma}")
        got = sbw.watermark_argmax(t, c, WIDE, gamma, delta, seeding, workspace=ws)
        assert_argmax_equal([g.cpu().numpy() for g in got],
                            oracle.watermark_argmax(x, ctx, WIDE, gamma, delta, seeding), f"greedy {B}x{V}")
        got = sbw.watermark_sample(t, c, WIDE, gamma, delta, s, seeding, 0.8, workspace=ws)
        assert_argmax_equal([g.cpu().numpy() for g in got],
                            oracle.watermark_sample(x, ctx, WIDE, gamma, delta, seeding, seeds, 0.8),
                            f"sample {B}x{V}")
        assert bool((ws == -5).all()) == short
    if B <= 7:
        got = sbw.watermark_argmax_noalloc(t, c, WIDE, 0.25, -1.5, seeding)
        assert_argmax_equal([g.cpu().numpy() for g in got],
                            oracle.watermark_argmax(x, ctx, WIDE, 0.25, -1.5, seeding), "no workspace")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_short_shard_winners(env, dtype):
    """Three shards of a row of 700 tokens: global ids, and the winners reduced to the row's."""
    torch, sbw, dev = env
    rng = np.random.default_rng(77)
    B, V = 40, 700
    x = (rng.standard_normal((B, V)) * 3).astype(np.float32)
    if dtype == "bf16":
        x = workloads.f32_to_bf16_bits(x)
    ctx = workloads.context_tokens(B, 2, V, rng)
    c = torch.from_numpy(np.ascontiguousarray(ctx, dtype=np.int32)).to(dev)
    t = _to_device(torch, dev, x)
    say(f"short shards {dtype}")
    parts = [sbw.watermark_argmax_shard(t[:, a:b], c, a, WIDE, 0.25, 2.0, "self_salt")
             for a, b in ((0, 61), (61, 350), (350, V))]
    tokens = np.stack([p[0].cpu().numpy() for p in parts])
    values = np.stack([p[1].cpu().numpy() for p in parts])
    best = values.argmax(axis=0)                      # the first of equal ones: the smaller id
    et, ev = oracle.watermark_argmax(x, ctx, WIDE, 0.25, 2.0, "self_salt")
    assert np.array_equal(tokens[best, np.arange(B)], et)
    assert np.array_equal(values[best, np.arange(B)].view(np.uint32), ev.view(np.uint32))
