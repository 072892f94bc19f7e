"""The entry points' native call path against their Python path.

An explicit `stream` argument takes the Python path, so each call is made both ways: the
outputs are the same bits, caller's buffers are the returned objects, and a call that the
Python path refuses raises the same error.
"""
import numpy as np
import pytest

from test_gpu_parity import WIDE, env  # noqa: F401

pytestmark = pytest.mark.gpu


def both(torch, f, *args, **kw):
    a = f(*args, **kw)
    b = f(*args, stream=torch.cuda.current_stream(), **kw)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert (x is None and y is None) or (x.dtype == y.dtype and x.shape == y.shape and
                                             torch.equal(x.view(torch.uint8), y.view(torch.uint8)))
    return a


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("B,V,pad,width,offset", [(1, 1, 0, 1, 0), (3, 4097, 3, 4, 0), (5, 9000, 0, 1, 1003)])
def test_logits_calls(env, dtype, B, V, pad, width, offset):
    torch, sbw, dev = env
    g = torch.Generator(device=dev).manual_seed(B + V)
    x = torch.randn((B, V + pad), generator=g, device=dev).to(getattr(torch, dtype))[:, :V]
    ctx = torch.randint(0, V + offset, (B, width), generator=g, device=dev, dtype=torch.int32)
    ctx = ctx[:, 0].contiguous() if width == 1 else ctx
    seeds = torch.randint(0, 1 << 62, (B,), generator=g, device=dev, dtype=torch.int64)
    cand = torch.randint(0, V, (B, 7), generator=g, device=dev, dtype=torch.int32)
    for seeding in ("context", "self_salt"):
        for key in (WIDE, -WIDE, WIDE + (1 << 64)):       # keys are taken modulo 2^64
            a, b = x.clone(), x.clone()
            assert sbw.watermark(a, ctx, key, 0.25, 2, seeding, v_offset=offset) is a
            sbw.watermark(b, ctx, key, 0.25, 2, seeding, stream=torch.cuda.current_stream(), v_offset=offset)
            assert torch.equal(a, b)
        sbw.watermark_candidates(a, ctx, cand, WIDE, 0.25, 2.0, seeding)
        sbw.watermark_candidates(b, ctx, cand, WIDE, 0.25, 2.0, seeding, stream=torch.cuda.current_stream())
        assert torch.equal(a, b)
        both(torch, sbw.watermark_argmax, x, ctx, WIDE, 0.25, 2.0, seeding, v_offset=offset)
        both(torch, sbw.watermark_argmax, x, ctx, WIDE, 0.25, 2.0, seeding, with_values=False, v_offset=offset)
        both(torch, sbw.watermark_sample, x, ctx, WIDE, 0.25, 2.0, seeds, seeding, 0.5, v_offset=offset)
        tokens = torch.empty(B, dtype=torch.int32, device=dev)
        values = torch.empty(B, dtype=torch.float32, device=dev)
        out = sbw.watermark_argmax(x, ctx, WIDE, 0.25, 2.0, seeding, tokens=tokens, values=values)
        assert out[0] is tokens and out[1] is values


def test_detect_calls(env):
    torch, sbw, dev = env
    g = torch.Generator(device=dev).manual_seed(5)
    t = torch.randint(0, 50, (9, 130), generator=g, device=dev, dtype=torch.int32)[:, :125]
    lengths = torch.randint(0, 126, (9,), generator=g, device=dev, dtype=torch.int32)
    for seeding in ("context", "self_salt"):
        assert len(both(torch, sbw.detect, t, WIDE, 0.25, seeding, width=2)) == 2
        for repeated in (False, True):
            both(torch, sbw.detect_ex, t, WIDE, 0.25, seeding, width=2, lengths=lengths, ignore_repeated=repeated)
    z = torch.empty(9, dtype=torch.float64, device=dev)
    assert sbw.detect(t, WIDE, 0.25, z=z)[1] is z


def test_refused_calls_and_other_forms(env):
    """What the Python path refuses or accepts beyond the plain form stays so."""
    torch, sbw, dev = env
    x = torch.zeros((4, 64), device=dev)
    p = torch.zeros(4, dtype=torch.int32, device=dev)
    t = torch.zeros((4, 64), dtype=torch.int32, device=dev)
    refused = [
        (lambda: sbw.watermark(x, p[:3], WIDE, 0.25, 2.0), ValueError),
        (lambda: sbw.watermark(x, p.cpu(), WIDE, 0.25, 2.0), ValueError),
        (lambda: sbw.watermark(x.t(), p, WIDE, 0.25, 2.0), ValueError),
        (lambda: sbw.watermark(x.double(), p, WIDE, 0.25, 2.0), TypeError),
        (lambda: sbw.watermark(x, p, WIDE, 0.25, 2.0, "bogus"), KeyError),
        (lambda: sbw.watermark(x, p, WIDE, 1.5, 2.0), sbw.SbwError),
        (lambda: sbw.watermark(x, p, WIDE, 0.25, 1e300), sbw.SbwError),
        (lambda: sbw.watermark(x, p, WIDE, 0.25, 2.0, v_offset=-1), sbw.SbwError),
        (lambda: sbw.watermark_argmax(x, p, WIDE, 0.25, 2.0, workspace=p), ValueError),
        (lambda: sbw.watermark_sample(x, p, WIDE, 0.25, 2.0, p), ValueError),
        (lambda: sbw.watermark_sample(x, p, WIDE, 0.25, 2.0, p.long(), inv_temperature=0.0), sbw.SbwError),
        (lambda: sbw.detect(t, WIDE, 0.0), sbw.SbwError),
        (lambda: sbw.detect(t, WIDE, 0.25, width=9), sbw.SbwError),
        (lambda: sbw.detect(t[:, ::2], WIDE, 0.25), ValueError),
        (lambda: sbw.detect_ex(t, WIDE, 0.25, scored=False), AttributeError),   # not a tensor
        (lambda: sbw.detect_ex(t, WIDE, 0.25, counts=False), AttributeError),
        (lambda: sbw.detect_ex(t, WIDE, 0.25, scored=p.long()), ValueError),
    ]
    for call, error in refused:
        with pytest.raises(error):
            call()
    assert torch.equal(x, torch.zeros_like(x))
    sbw.watermark(torch.nn.Parameter(x.clone(), requires_grad=False), p, np.int64(7), np.float32(0.25),
                  np.float64(2.0), sbw.SEED_SELF_SALT)
    assert sbw.detect(t[:0], WIDE, 0.25)[0].shape == (0,)
    assert sbw.watermark(x[:0], p[:0], WIDE, 0.25, 2.0).shape == (0, 64)
    side = torch.cuda.Stream()
    a, b = x.clone(), x.clone()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                         # the current stream, not the default one
        sbw.watermark(a, p, WIDE, 0.25, 2.0)
    side.synchronize()
    sbw.watermark(b, p, WIDE, 0.25, 2.0)
    assert torch.equal(a, b)
