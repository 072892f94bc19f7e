"""GPU parity of the self-salt split-term slab kernel (fp32 and bf16, window of one token).

Large self-salt launches take a kernel that draws each column's self-term block once
per slab of 12 rows (8, then, fp32, 6 for launches that taller slabs would leave with too
few workgroups) and queues in LDS only the (row, token) pairs whose row term is the
smaller one.  Every case here is sized to take that kernel (the launch rule is
mirrored in `slab_rows`, with its figures read from the kernel source, and asserted),
and is compared with the oracle bit for bit:
  * slabs cut short (B not a multiple of 12), a row tail (V mod 4 != 0), the last
    workgroup tile partly past the row, padded rows, rows off 16 bytes;
  * special values (NaNs with payloads, infinities, signed zeros, subnormals);
  * gamma from tiny to 1 (every token green), both key shapes, both signs of delta;
  * a vocabulary shard whose first token id is a multiple of 4, as one of 8
    tensor-parallel heads of the 152064-token vocabulary holds it, and shards that start
    inside a vector of token ids (columns before the first whole one), in every slab height;
  * two launches back to back, the second smaller (nothing a launch leaves in LDS
    changes the next one);
  * more slabs than the grid's y dimension holds (workgroups that take two).
The c4 configurations at full size (B = 256 and 1024) take this kernel too and are
checked in test_gpu_parity.py.
"""
import pathlib
import re

import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import (KEY, WIDE, _from_device, _to_device, assert_logits_equal, env,  # noqa: F401
                             say, special_logits)

pytestmark = pytest.mark.gpu

SLAB_ROWS = 12
SOURCE = pathlib.Path(__file__).resolve().parents[1] / "paper_2609_03844_amd" / "csrc" / "sbw_kernels.hip"


def knob(name):
    return int(re.search(rf"#define {name} (\d+)", SOURCE.read_text()).group(1))


def slab_rows(B, V, dtype="f32", start=0):
    """The launch rule of the self-salt watermark, window of one token, for columns
    start .. start + V - 1: the slab height the launch takes, or 0 for the row kernel.  Tiles
    are of 256 whole 16-byte vectors whose first token id is a multiple of their tokens."""
    if V <= 256:
        return 0                          # one token per lane
    per = 4 if dtype == "f32" else 8
    head = min(-start % per, V)
    tiles = -(-((V - head) // per) // 256)
    heights = ([(12, knob("SBW_SLAB12_MIN_GROUPS")), (8, knob("SBW_SLAB_MIN_GROUPS")),
                (6, knob("SBW_SLAB_MIN_GROUPS"))] if dtype == "f32"
               else [(12, knob("SBW_SLAB12_MIN_GROUPS")), (8, knob("SBW_SLAB_BF16_MIN_GROUPS"))])
    for rows, least in heights:
        if tiles * -(-B // rows) >= least:
            return rows
    return 0


def takes_slab(B, V):
    return slab_rows(B, V) == SLAB_ROWS


def run(env, x, prev, key, gamma, delta, stride=None, v_offset=None, offset=0):
    """Watermarks x in a device buffer of rows `stride` elements apart (by default V), the
    first `offset` elements into it.  Returns the rows and the elements around them."""
    torch, sbw, dev = env
    B, V = x.shape
    stride = stride or V
    dt = torch.bfloat16 if x.dtype == np.uint16 else torch.float32
    base = torch.zeros(offset + B * stride, dtype=dt, device=dev)
    rows = base[offset:].view(B, stride)
    rows[:, :V] = _to_device(torch, dev, x)
    p = torch.from_numpy(prev).to(dev)
    if v_offset is None:
        sbw.watermark(rows[:, :V], p, key, gamma, delta, "self_salt")
    else:
        sbw.watermark_shard(rows[:, :V], p, v_offset, key, gamma, delta, "self_salt")
    torch.cuda.synchronize()
    out = _from_device(torch, rows)
    around = np.concatenate([_from_device(torch, base[:offset]), out[:, V:].ravel()])
    return out[:, :V], around


def shard_expect(x, prev, start, key, gamma, delta):
    """The oracle's membership of tokens start .. start + n - 1 in each row, and its bias."""
    B, n = x.shape
    green = oracle.is_green_many(key, np.repeat(prev, n), np.tile(np.arange(start, start + n), B), gamma,
                                 "self_salt").reshape(B, n)
    many = oracle.bias_bf16_many if x.dtype == np.uint16 else oracle.bias_f32_many
    return np.where(green, many(x, delta), x)


@pytest.mark.parametrize("B,V,stride", [
    (4501, 8199, None),      # slab of 1 row at the end, V mod 4 = 3, 2049 vectors (tile of 1)
    (3600, 10241, 10248),    # whole slabs, padded rows, V mod 4 = 1
    (2125, 16390, None),     # V mod 4 = 2, last tile partly past the row
    (893, 40000, 40004),     # whole vectors, padded rows, slab of 5 rows at the end
    (893, 40000, 40001),     # the same, rows off 16 bytes
])
def test_slab_shapes(env, B, V, stride):
    assert takes_slab(B, V)
    rng = np.random.default_rng(77 + B + V)
    x = special_logits(rng, B, V, "f32")
    prev = rng.integers(0, 1 << 31, B).astype(np.int32)
    prev[:3] = [0, -1, 2**31 - 1]
    say(f"slab shapes B={B} V={V} stride={stride}")
    got, pad = run(env, x, prev, WIDE, 0.25, 2.0, stride)
    assert_logits_equal(got, oracle.watermark(x, prev, WIDE, 0.25, 2.0, "self_salt"),
                        f"B={B} V={V}")
    assert not pad.any(), "elements around the rows were written"


@pytest.mark.parametrize("gamma,delta,key", [
    (0.25, 2.0, KEY),
    (0.5, -3.0, WIDE),
    (1e-9, 8.0, WIDE),       # almost no token green
    (1.0 - 1e-10, 1.0, KEY),
    (1.0, 4.0, WIDE),        # every token green
])
def test_slab_parameters(env, gamma, delta, key):
    B, V = 2762, 12292
    assert takes_slab(B, V)
    rng = np.random.default_rng(int(gamma * 1e6) + int(delta * 10) + 5)
    x = rng.standard_normal((B, V)).astype(np.float32)
    prev = rng.integers(0, V, B).astype(np.int32)
    say(f"slab parameters gamma={gamma} delta={delta}")
    got, _ = run(env, x, prev, key, gamma, delta)
    assert_logits_equal(got, oracle.watermark(x, prev, key, gamma, delta, "self_salt"),
                        f"gamma={gamma} delta={delta}")


def test_slab_shard(env):
    """Columns [57024, 57024 + 19008) of a 152064-token vocabulary (one of 8 shards) at
    B = 1900: token ids from 57024, the draws those of the full row."""
    a, n, V, B = 57024, 19008, 152064, 1900
    assert takes_slab(B, n)
    rng = np.random.default_rng(4242)
    x = rng.standard_normal((B, n)).astype(np.float32) * np.float32(3)
    prev = rng.integers(0, V, B).astype(np.int32)
    say("slab shard 57024+19008, B=1900")
    got, _ = run(env, x, prev, WIDE, 0.25, 2.0, v_offset=a)
    assert_logits_equal(got, shard_expect(x, prev, a, WIDE, 0.25, 2.0), "shard")


@pytest.mark.parametrize("dtype,B,n,start,rows,offset,pad", [
    ("f32", 2129, 16391, 57025, 12, 0, 0),    # 3 columns before the first vector, 4097 vectors
    ("f32", 36003, 258, 1003, 12, 1, 3),      # one column before, one after; a slab of 3 rows
    ("f32", 36001, 261, 2, 12, 0, 1),         # 2 before, 3 after
    ("f32", 16005, 307, 1001, 8, 3, 2),       # 8-row slabs, a last one of 5 rows
    ("f32", 12005, 1027, 6, 6, 2, 0),         # 6-row slabs, a last one of 5 rows, 256 vectors
    ("bf16", 36005, 301, 57027, 12, 1, 4),    # 5 before, none after
    ("bf16", 36000, 270, 9, 12, 0, 1),        # 7 before, 7 after
    ("bf16", 18001, 2060, 4, 12, 3, 0),       # 4 before, 257 vectors
    ("bf16", 21605, 261, 2, 8, 1, 2),         # 8-row slabs, a last one of 5 rows; 6 before, 7 after
])
def test_slab_shard_inside_a_vector(env, dtype, B, n, start, rows, offset, pad):
    """Shards whose first token id is not a multiple of a vector's tokens."""
    assert start % (4 if dtype == "f32" else 8) and slab_rows(B, n, dtype, start) == rows
    rng = np.random.default_rng(B + n + start)
    x = special_logits(rng, B, n, dtype)
    prev = rng.integers(0, 1 << 31, B).astype(np.int32)
    say(f"slab shard inside a vector {dtype} {start}+{n}, B={B}")
    got, around = run(env, x, prev, WIDE, 0.4, 1.5, n + pad, v_offset=start, offset=offset)
    assert_logits_equal(got, shard_expect(x, prev, start, WIDE, 0.4, 1.5), f"{dtype} {start}+{n}")
    assert not around.any(), "elements around the rows were written"


def test_slab_twice_in_a_row(env):
    """Two launches back to back, the second smaller, on fresh inputs each: nothing a
    launch leaves in LDS or in the logits changes the next one's result."""
    rng = np.random.default_rng(99)
    for B, V in ((3000, 12300), (2900, 12299)):
        assert takes_slab(B, V)
        x = rng.standard_normal((B, V)).astype(np.float32)
        prev = rng.integers(0, V, B).astype(np.int32)
        say(f"slab twice B={B} V={V}")
        got, _ = run(env, x, prev, KEY, 0.25, 2.0)
        assert_logits_equal(got, oracle.watermark(x, prev, KEY, 0.25, 2.0, "self_salt"),
                            f"B={B} V={V}")


def test_slab_grid_stride(env):
    """More slabs than the 65535 workgroups of the grid's y dimension: some workgroups
    take a second slab (800003 rows of 258 logits: a 2-logit row tail, a last slab of 11
    rows).  The oracle checks the first rows, those around the second slabs and the last."""
    torch, sbw, dev = env
    B, V = 800003, 258
    assert takes_slab(B, V) and -(-B // SLAB_ROWS) > 65535
    rng = np.random.default_rng(5150)
    x = torch.randn((B, V), generator=torch.Generator(device=dev).manual_seed(5150), device=dev)
    prev = rng.integers(0, 1 << 20, B).astype(np.int32)
    second = 65000 * SLAB_ROWS
    pick = np.r_[0:3000, second:second + 9000, B - 9000:B]
    at = torch.from_numpy(pick).to(dev)
    before = x[at].cpu().numpy()
    say(f"slab grid stride B={B} V={V}")
    sbw.watermark(x, torch.from_numpy(prev).to(dev), WIDE, 0.25, 2.0, "self_salt")
    assert_logits_equal(x[at].cpu().numpy(), oracle.watermark(before, prev[pick], WIDE, 0.25, 2.0, "self_salt"),
                        "grid stride")


@pytest.mark.parametrize("B,V", [
    (128, 128256),    # whole 8-row slabs
    (131, 128255),    # a last slab of 3 rows, V mod 4 = 3
])
def test_slab_eight_rows(env, B, V):
    """Launches that 12-row slabs would leave with too few workgroups (here under 2000;
    below 3000 as well) take 8-row ones."""
    assert slab_rows(B, V) == 8
    rng = np.random.default_rng(808 + B)
    x = special_logits(rng, B, V, "f32")
    prev = rng.integers(0, V, B).astype(np.int32)
    say(f"slab 8 rows B={B} V={V}")
    got, _ = run(env, x, prev, WIDE, 0.25, 2.0)
    assert_logits_equal(got, oracle.watermark(x, prev, WIDE, 0.25, 2.0, "self_salt"),
                        f"B={B} V={V}")


@pytest.mark.parametrize("B,V", [
    (96, 128256),     # whole 6-row slabs
    (101, 128255),    # a last slab of 5 rows, V mod 4 = 3
    (80, 152064),
])
def test_slab_six_rows(env, B, V):
    """Launches that 8-row slabs would leave with too few workgroups take 6-row ones."""
    assert slab_rows(B, V) == 6
    rng = np.random.default_rng(606 + B)
    x = special_logits(rng, B, V, "f32")
    prev = rng.integers(0, V, B).astype(np.int32)
    say(f"slab 6 rows B={B} V={V}")
    got, _ = run(env, x, prev, KEY, 0.5, -2.0)
    assert_logits_equal(got, oracle.watermark(x, prev, KEY, 0.5, -2.0, "self_salt"),
                        f"B={B} V={V}")


@pytest.mark.parametrize("B,V,stride,offset,rows", [
    (36001, 263, None, 0, 12),      # V mod 8 = 7, rows off 16 bytes, a last slab of 1 row
    (36007, 264, 272, 0, 12),       # whole vectors, padded aligned rows, a last slab of 7 rows
    (18007, 2059, 2064, 0, 12),     # 257 vectors (tile of 1), V mod 8 = 3, padded aligned rows
    (18000, 2057, None, 3, 12),     # the same off 16 bytes, whole slabs
    (3600, 20483, None, 0, 12),     # 10 tiles
    (21603, 264, None, 0, 8),       # 8-row slabs, a last one of 3 rows
    (400, 152064, None, 0, 8),
])
def test_slab_bf16(env, B, V, stride, offset, rows):
    """bf16 logits: 8 tokens a vector, two Philox counters a lane, 8 map bytes a row."""
    assert slab_rows(B, V, "bf16") == rows
    rng = np.random.default_rng(1616 + B + V)
    x = special_logits(rng, B, V, "bf16")
    prev = rng.integers(0, 1 << 31, B).astype(np.int32)
    prev[:2] = [0, -1]
    say(f"slab bf16 B={B} V={V} stride={stride} offset={offset}")
    got, pad = run(env, x, prev, WIDE, 0.25, 2.0, stride, offset=offset)
    assert_logits_equal(got, oracle.watermark(x, prev, WIDE, 0.25, 2.0, "self_salt"),
                        f"bf16 B={B} V={V}")
    assert not pad.any(), "elements around the rows were written"


@pytest.mark.parametrize("B,V,stride", [
    (1600, 20483, None),      # rows off 16 bytes, V mod 8 = 3
    (1607, 20480, 20488),     # padded rows
    (256, 152064, None),      # the c4 shape in bf16
    (263, 152061, 152064),    # V mod 8 = 5
    (192, 152064, None),
    (197, 152061, 152064),
])
def test_bf16_below_the_slab_line(env, B, V, stride):
    """bf16 launches of too few workgroups for slabs take the row kernel."""
    assert slab_rows(B, V, "bf16") == 0
    rng = np.random.default_rng(1616 + B + V)
    x = special_logits(rng, B, V, "bf16")
    prev = rng.integers(0, 1 << 31, B).astype(np.int32)
    prev[:2] = [0, -1]
    say(f"bf16 below the slab line B={B} V={V} stride={stride}")
    got, pad = run(env, x, prev, WIDE, 0.25, 2.0, stride)
    assert_logits_equal(got, oracle.watermark(x, prev, WIDE, 0.25, 2.0, "self_salt"),
                        f"bf16 B={B} V={V}")
    assert not pad.any(), "elements around the rows were written"


@pytest.mark.parametrize("gamma,delta,key", [
    (0.5, -3.0, KEY),
    (1e-9, 8.0, WIDE),
    (1.0 - 1e-10, 1.0, KEY),
    (1.0, 4.0, WIDE),
])
def test_slab_bf16_parameters(env, gamma, delta, key):
    B, V = 36003, 269
    assert slab_rows(B, V, "bf16") == 12
    rng = np.random.default_rng(int(gamma * 1e6) + int(delta * 10) + 7)
    x = special_logits(rng, B, V, "bf16")
    prev = rng.integers(0, 1 << 31, B).astype(np.int32)
    say(f"slab bf16 parameters gamma={gamma} delta={delta}")
    got, _ = run(env, x, prev, key, gamma, delta)
    assert_logits_equal(got, oracle.watermark(x, prev, key, gamma, delta, "self_salt"),
                        f"bf16 gamma={gamma} delta={delta}")


def test_slab_bf16_shard(env):
    """A bf16 vocabulary shard whose first token id is a multiple of 8 (not of 16)."""
    a, n, V, B = 57024 + 8, 264, 152064, 36013
    assert slab_rows(B, n, "bf16", a) == 12
    rng = np.random.default_rng(4343)
    x = workloads.f32_to_bf16_bits(rng.standard_normal((B, n)).astype(np.float32) * np.float32(2))
    prev = rng.integers(0, V, B).astype(np.int32)
    say(f"slab bf16 shard {a}+{n}, B={B}")
    got, _ = run(env, x, prev, KEY, 0.5, -1.5, v_offset=a)
    assert_logits_equal(got, shard_expect(x, prev, a, KEY, 0.5, -1.5), "bf16 shard")


def test_launch_rule_cases():
    """The c4 configurations take 12-row slabs, B = 160-240 of 152064 tokens and B = 128
    of 128256 8-row ones, B = 96 6-row ones; c3 and small batches take the row kernel.
    bf16 takes 12-row slabs from about B = 500, 8-row ones from about 300."""
    assert slab_rows(256, 152064) == 12 and slab_rows(1024, 152064) == 12
    assert slab_rows(160, 152064) == 8 and slab_rows(240, 152064) == 8
    assert slab_rows(128, 128256) == 8 and slab_rows(96, 128256) == 6
    assert slab_rows(64, 128256) == 0 and slab_rows(16, 152064) == 0
    assert slab_rows(1024, 152064, "bf16") == 12
    assert slab_rows(512, 152064, "bf16") == 12 and slab_rows(400, 152064, "bf16") == 8
    assert slab_rows(256, 152064, "bf16") == 0
