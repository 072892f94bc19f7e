"""GPU parity of the watermark on rows and shards that start anywhere.

Logits move in 16-byte vectors (self-salt: 4-token quads) from any element address, with
the columns before the first whole Philox block and after the last one taken one by one.
Small launches, and rows of at most 256 columns, take one token per lane.  The cases cover
every start modulo 8 of a shard, rows shorter than a vector, rows one column either side of
whole vectors and tiles, odd row strides and base offsets, windows of 1-8 tokens (each its
own self-salt kernel), one and two quads per lane, workgroups that take several rows, and
both sides of the lines between one token per lane and vectors.  Logits bit for bit against
the oracle, and nothing outside the shard's columns may change.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import WIDE, assert_logits_equal, env, say, special_logits, _from_device, _to_device  # noqa: F401

pytestmark = pytest.mark.gpu


def check(env, dtype, seeding, width, B, start, n, offset=0, pad=0, gamma=0.25, delta=2.0):
    """A shard of columns start .. start + n - 1, in rows of n + pad elements that begin
    `offset` elements into a buffer."""
    torch, sbw, dev = env
    rng = np.random.default_rng(B * 31 + start * 7 + n + width + offset)
    full = special_logits(rng, B, start + n, "f32")
    if dtype == "bf16":
        full = workloads.f32_to_bf16_bits(full)
    ctx = workloads.context_tokens(B, width, start + n, rng)
    stride = n + pad
    base = np.zeros(offset + B * stride + 16, dtype=full.dtype)
    base[:] = 3
    rows = np.lib.stride_tricks.as_strided(base[offset:], shape=(B, n),
                                           strides=(stride * base.itemsize, base.itemsize))
    rows[...] = full[:, start:]
    expect = base.copy()
    np.lib.stride_tricks.as_strided(expect[offset:], shape=(B, n),
                                    strides=(stride * base.itemsize, base.itemsize))[...] = \
        oracle.watermark_w(full, ctx, WIDE, gamma, delta, seeding)[:, start:]
    t = _to_device(torch, dev, base)
    c = torch.from_numpy(np.ascontiguousarray(ctx, dtype=np.int32)).to(dev)
    what = f"{dtype} {seeding} h={width} B={B} start={start} n={n} offset={offset} pad={pad}"
    say("any alignment " + what)
    sbw.watermark_shard(t[offset:offset + B * stride].view(B, stride)[:, :n], c, start, WIDE, gamma, delta,
                        seeding)
    torch.cuda.synchronize()
    assert_logits_equal(_from_device(torch, t)[None], expect[None], what)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seeding", ["context", "self_salt"])
@pytest.mark.parametrize("width", [1, 3, 8])
def test_every_start_and_short_rows(env, dtype, seeding, width):
    for start in range(9):
        for n in (1, 2, 5, 8, 9, 15, 23, 1027, 4101):
            check(env, dtype, seeding, width, 5, start, n, offset=start % 3, pad=n % 4)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seeding", ["context", "self_salt"])
@pytest.mark.parametrize("width", [1, 3, 8])
def test_every_start_with_vectors(env, dtype, seeding, width):
    """Rows of more than 256 columns, more logits than one token per lane takes."""
    for start in range(9):
        for n in (1027, 4101):
            check(env, dtype, seeding, width, 440000 // n, start, n, offset=start % 3, pad=n % 4)
    for start, n in ((0, 257), (3, 263), (5, 511)):
        check(env, dtype, seeding, width, 860000 // n, start, n, offset=1, pad=1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seeding,width,whole,edges", [
    ("context", 4, 8 << 15, 10 << 15), ("self_salt", 1, 8 << 15, 13 << 15), ("self_salt", 2, 6 << 15, 12 << 15),
    ("self_salt", 4, 5 << 15, 9 << 15), ("self_salt", 5, 4 << 15, 5 << 15)])
def test_either_side_of_one_token_per_lane(env, dtype, seeding, width, whole, edges):
    """The launches on both sides of each line: most logits of rows of whole vectors, of rows
    with edge columns and of such rows of at most 512 columns; rows of 256 and 257 columns."""
    for n, most in ((1024, whole), (1023, edges), (511, 2 * edges)):
        for B in (most // n, most // n + 1):
            check(env, dtype, seeding, width, B, 0, n, pad=0 if n == 1024 else 1)
    for n in (255, 256, 257):
        check(env, dtype, seeding, width, 4000, 1, n)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("seeding", ["context", "self_salt"])
@pytest.mark.parametrize("n", [4095, 4096, 4097, 8191, 8193])
def test_tile_edges(env, dtype, seeding, n):
    for start, offset, pad in [(0, 0, 0), (0, 1, 1), (1003, 0, 3), (1004, 5, 0)]:
        for B in (37, 110):                  # one token per lane, or vectors; vectors
            check(env, dtype, seeding, 2, B, start, n, offset, pad)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 6, 7, 8])
def test_self_salt_rows_in_turn(env, dtype, width):
    """Enough workgroups for two quads per lane and several rows each (B not a multiple)."""
    check(env, dtype, "self_salt", width, 67, 0, 30003)
    check(env, dtype, "self_salt", width, 143, 1025, 10241, offset=1, pad=2, delta=-1.5)


def test_bf16_slab(env):
    """bf16, window of one token: 12-row slabs (10 tiles x 501 workgroups)."""
    check(env, "bf16", "self_salt", 1, 6005, 0, 20477, pad=2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_context_whole_rows_per_xcd_with_edges(env, dtype):
    """Launches large enough for whole rows per XCD, whose rows have single columns."""
    check(env, dtype, "context", 4, 512 if dtype == "f32" else 1024, 3, 131079)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,n", [(299, 2051), (300, 2051), (301, 5003), (3000, 301), (4999, 517), (40003, 270)])
def test_context_edges_behind_and_between_the_tiles(env, dtype, B, n):
    """From 300 rows the edge columns' grid rows are spread between the tiles': one of them and
    many, each with one and with many tiles, and rows that are not a multiple of their distance."""
    check(env, dtype, "context", 2, B, 3, n, offset=1, pad=1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("B,start,n,pad", [(3, 1, 1, 0), (5, 3, 4, 1), (4, 5, 15, 0), (3, 7, 4096, 3),
                                           (2, 2, 12290, 1), (200, 1003, 40969, 2)])
def test_decode_from_any_column(env, dtype, sample, B, start, n, pad):
    """Greedy decoding and sampling of a shard: token and value bit for bit, with the row's
    winner in turn before, inside and after its whole vectors."""
    torch, sbw, dev = env
    rng = np.random.default_rng(B + start + n)
    x = special_logits(rng, B, start + n, "f32")
    x[~np.isfinite(x)] = 0.0
    for b in range(B):
        x[b, start + [0, n - 1, n // 2][b % 3]] = 1e4
    full = workloads.f32_to_bf16_bits(x) if dtype == "bf16" else x
    shard = np.zeros((B, n + pad), dtype=full.dtype)
    shard[:, :n] = full[:, start:]
    ctx = workloads.context_tokens(B, 2, start + n, rng)
    seeds = rng.integers(0, 2**63, B, dtype=np.int64)
    hidden = full.copy()      # the whole row with the columns before the shard out of the running
    hidden[:, :start] = workloads.f32_to_bf16_bits(np.float32([-1e30]))[0] if dtype == "bf16" else -1e30
    t = _to_device(torch, dev, shard)[:, :n]
    c = torch.from_numpy(np.ascontiguousarray(ctx, dtype=np.int32)).to(dev)
    for seeding in ("context", "self_salt"):
        say(f"decode from any column {dtype} {seeding} sample={sample} B={B} start={start} n={n} pad={pad}")
        if sample:
            got = sbw.watermark_sample(t, c, WIDE, 0.25, 2.0, torch.from_numpy(seeds).to(dev), seeding, 0.7,
                                       v_offset=start)
            expect = oracle.watermark_sample(hidden, ctx, WIDE, 0.25, 2.0, seeding, seeds.view(np.uint64), 0.7)
        else:
            got = sbw.watermark_argmax(t, c, WIDE, 0.25, 2.0, seeding, v_offset=start)
            expect = oracle.watermark_argmax(hidden, ctx, WIDE, 0.25, 2.0, seeding)
        assert np.array_equal(got[0].cpu().numpy(), expect[0])
        assert np.array_equal(got[1].cpu().numpy().view(np.uint32), expect[1].view(np.uint32))
