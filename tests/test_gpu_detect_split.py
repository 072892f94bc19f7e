"""GPU parity of detection where several waves or workgroups share a sequence.

Few sequences are scored by up to 16 waves each, and sequences of more than 64 chunks of
64 positions by several workgroups, whose counts meet in the sequence's z slot.  The
cases sit on both sides of every line of that choice: one chunk and two, 64 chunks and 65,
the batches at which fewer waves or splits are taken (and the first that take one wave
per sequence, for two, three and four chunks), a last pass that only some waves have, texts that end before a split's
first position.  Windows of 1, 2, 5 and 8 tokens share their hashed terms through LDS
(self-salt) or not.  Counts and scored counts equal the oracle's, z within 1e-6 relative;
every case runs twice on the same output buffers, so a slot left over from the first run
would show.
"""
import numpy as np
import pytest

import oracle
from test_gpu_detect_ex import assert_ex_equal
from test_gpu_parity import WIDE, env, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seeding", ["context", "self_salt"])
@pytest.mark.parametrize("width", [1, 2, 5, 8])
@pytest.mark.parametrize("N,L", [(1, 72), (3, 137), (2, 4105), (2, 4300), (9, 4300), (33, 4170), (7, 16390),
                                 (513, 260), (1025, 200), (2049, 75), (255, 130), (256, 130), (300, 180),
                                 (767, 250), (768, 250), (1000, 300), (600, 600), (1500, 420)])
def test_detect_split(env, seeding, width, N, L):
    torch, sbw, dev = env
    rng = np.random.default_rng(900 + width + N + L)
    tok = rng.integers(0, 128256, (N, L)).astype(np.int32)
    lengths = rng.integers(0, L + 1, N).astype(np.int32)
    lengths[0] = L
    if N > 4:
        lengths[1:4] = [0, width, width + 1]
    host = np.full((N, L + 3), 7, dtype=np.int32)
    host[:, :L] = tok
    t = torch.from_numpy(host).to(dev)[:, :L]
    lens = torch.from_numpy(lengths).to(dev)
    out = dict(counts=torch.full((N,), -1, dtype=torch.int32, device=dev),
               scored=torch.full((N,), -1, dtype=torch.int32, device=dev),
               z=torch.full((N,), float("nan"), dtype=torch.float64, device=dev))
    expect = oracle.detect_ex(tok, width, WIDE, 0.25, seeding, lengths=lengths)
    say(f"detect split {seeding} h={width} N={N} L={L}")
    for _ in range(2):
        sbw.detect_ex(t, WIDE, 0.25, seeding, width=width, lengths=lens, **out)
        torch.cuda.synchronize()
        assert_ex_equal(tuple(out[k].cpu().numpy() for k in ("counts", "scored", "z")), expect,
                        f"{seeding}/{width}/{N}x{L}")
