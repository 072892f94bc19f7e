"""Rows with single columns, narrow rows and short rows keep near the time of plain ones.

Results are the same whichever kernel takes such a launch, so these compare times: what each
case must not cost, against a launch of whole vectors or of the plain watermark.  The limits lie
between the ratios measured with the present launches and with vectors, segments and a
workgroup column for the single columns throughout, which the comments give.
"""
import pytest

from test_gpu_decode_bound import shortest_us
from test_gpu_parity import WIDE, env, say  # noqa: F401

pytestmark = pytest.mark.gpu


def rows(torch, dev, B, V, dtype):
    g = torch.Generator(device=dev).manual_seed(B + V)
    return (torch.randn((B, V), generator=g, device=dev).to(getattr(torch, dtype)),
            torch.randint(0, V, (B,), generator=g, device=dev, dtype=torch.int32),
            torch.randint(0, 1 << 62, (B,), generator=g, device=dev, dtype=torch.int64))


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_narrow_and_odd_rows(env, dtype):
    torch, sbw, dev = env

    def watermark(B, V, seeding):
        x, prev, _ = rows(torch, dev, B, V, dtype)
        return shortest_us(torch, lambda: sbw.watermark(x, prev, WIDE, 0.25, 2.0, seeding))

    def sample(B, V):
        x, prev, seeds = rows(torch, dev, B, V, dtype)
        ws = torch.empty(sbw.argmax_workspace_size(B, V), dtype=torch.int64, device=dev)
        out = torch.empty(B, dtype=torch.int32, device=dev), torch.empty(B, dtype=torch.float32, device=dev)
        return shortest_us(torch, lambda: sbw.watermark_sample(x, prev, WIDE, 0.25, 2.0, seeds, "context",
                                                               tokens=out[0], scores=out[1], workspace=ws))

    odd = watermark(1000, 2001, "self_salt") / watermark(1000, 2000, "self_salt")
    narrow = watermark(20000, 37, "context") / watermark(20000, 256, "context")
    short = sample(5000, 100) / watermark(5000, 256, "context")
    say(f"row time {dtype}: odd {odd:.2f}, narrow {narrow:.2f}, short {short:.2f}")
    assert odd < 1.3         # 1.04-1.09; with a workgroup column for the single columns 1.55
    assert narrow < 1.25     # 0.82-0.84; with vectors 1.8
    assert short < 2.3       # 1.06-1.16; in segments 4.8-5.8
