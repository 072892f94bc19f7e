"""The rising bound of the fused decoding pass.

Tokens are queued while they may still reach a wave's best score, and scoring a full queue
raises what the later ones have to reach.  Where delta is large against the logits' spread
nearly every token passes the first test, so without that rise nearly every token's colour is
drawn; the same holds for a bound of +inf that is not compared as such.  The results are the
same either way, so one test compares times: decoding such logits against decoding logits of
a wide spread in the same launch shape.  The limits lie between the ratios measured with the
rise and with a bound fixed per sub-batch (64 x 128256: greedy fp32 1.5 / 3.6, bf16 1.7 / 3.4,
sampling fp32 1.4 / 3.2, bf16 2.2 / 3.0; with infinities 1.0 / 1.9-2.1 in all four).  The other
compares results, bit for bit with the oracle, on rows that fill the queue many times over
with every kind of value the raised bound meets.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_argmax import assert_argmax_equal, run_argmax
from test_gpu_parity import WIDE, env, say  # noqa: F401
from test_gpu_sample import run_sample, seeds_for

pytestmark = pytest.mark.gpu


def shortest_us(torch, call):
    """Shortest time of a call over several replays of a graph of 20."""
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(20):
            call()
    times = []
    for _ in range(10):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        g.replay()
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 50.0)
    return min(times)


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("sample", [False, True])
def test_large_delta_and_infinities_stay_near_the_ordinary_time(env, dtype, sample):
    torch, sbw, dev = env
    B, V = 64, 128256
    g = torch.Generator(device=dev).manual_seed(5)
    ctx = torch.randint(0, V, (B,), generator=g, device=dev, dtype=torch.int32)
    seeds = torch.randint(0, 1 << 62, (B,), generator=g, device=dev, dtype=torch.int64)
    ws = torch.empty(sbw.argmax_workspace_size(B, V), dtype=torch.int64, device=dev)
    out = torch.empty(B, dtype=torch.int32, device=dev), torch.empty(B, dtype=torch.float32, device=dev)
    noise = torch.randn((B, V), generator=g, device=dev)

    def us(x, delta):
        x = x.to(getattr(torch, dtype))
        if sample:
            return shortest_us(torch, lambda: sbw.watermark_sample(
                x, ctx, WIDE, 0.25, delta, seeds, "self_salt", tokens=out[0], scores=out[1], workspace=ws))
        return shortest_us(torch, lambda: sbw.watermark_argmax(
            x, ctx, WIDE, 0.25, delta, "self_salt", tokens=out[0], values=out[1], workspace=ws))

    wide = us(noise * 3.0, 2.0)
    narrow = us(noise * 2.0, 8.0)
    inf = noise * 3.0
    inf[:, ::4099] = float("inf")
    inf = us(inf, 2.0)
    say(f"decode bound {dtype} sample={sample}: {wide:.1f} us, narrow {narrow:.1f}, inf {inf:.1f}")
    assert narrow < (2.55 if sample and dtype == "bfloat16" else 2.3) * wide
    assert inf < 1.45 * wide


def full_queue_rows(rng, V):
    """Rows nearly all of whose tokens pass the first test, by what the exact scores hold."""
    x = rng.standard_normal((14, V)).astype(np.float32)
    x[1] *= 0.01                                   # ties in bf16
    x[2] = 0.5                                     # all equal
    x[3] = -3e38                                   # sums with delta and bounds near -FLT_MAX
    x[4] = 3e38
    x[5] = np.float32(3e38) * (1 + x[5] * np.float32(0.02))      # some above FLT_MAX / bf16's
    x[6] = -np.abs(x[6]) * np.float32(1e38)
    x[7, ::97] = np.inf                            # a bound of +inf, ties of it
    x[8, 5::977] = np.nan                          # NaN among the exact scores
    x[9, V - 3] = np.nan
    x[10] = -np.inf
    x[10, V // 2] = -3.4e38
    x[11] = np.linspace(-1.0, 1.0, V)              # later tokens always better
    x[12] = np.linspace(1.0, -1.0, V)
    x[13] *= np.float32(1e-40)                     # subnormal
    return x


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seeding,width", [("context", 4), ("self_salt", 1), ("self_salt", 8)])
@pytest.mark.parametrize("V,tile", [(12290, 1), (16384, 20), (40003, 20)])   # half- and full-width segments
def test_many_queue_rounds(env, dtype, seeding, width, V, tile):
    rng = np.random.default_rng(V + width)
    with np.errstate(over="ignore"):
        x = full_queue_rows(rng, V)
    if dtype == "bf16":
        x = workloads.f32_to_bf16_bits(x)
    B = x.shape[0]
    ctx = workloads.context_tokens(B, width, V, rng)
    seeds = seeds_for(rng, B)
    tiled = [np.tile(a, (tile,) + (1,) * (a.ndim - 1)) for a in (x, ctx, seeds)]
    for gamma, delta in ((0.25, 4.0), (0.02, 8.0), (0.5, -6.0), (0.25, 3e38), (1.0, 1e36)):
        say(f"queue rounds {dtype} {seeding} h={width} V={V} gamma={gamma} delta={delta}")
        t, v = run_argmax(env, tiled[0], tiled[1], WIDE, gamma, delta, seeding)
        expect = oracle.watermark_argmax(x, ctx, WIDE, gamma, delta, seeding)
        for k in range(tile):
            assert_argmax_equal((t[k * B:(k + 1) * B], v[k * B:(k + 1) * B]), expect, f"greedy {gamma}/{delta}")
        t, v = run_sample(env, tiled[0], tiled[1], tiled[2], WIDE, gamma, delta, seeding, 0.7)
        expect = oracle.watermark_sample(x, ctx, WIDE, gamma, delta, seeding, seeds, 0.7)
        for k in range(tile):
            assert_argmax_equal((t[k * B:(k + 1) * B], v[k * B:(k + 1) * B]), expect, f"sample {gamma}/{delta}")
