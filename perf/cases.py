"""The performance cases of the watermark library: what its users have it do, one call each.

A decode step hands a batch of next-token logits to ``watermark`` (in place, then the
caller's own sampler), or straight to the fused ``watermark_argmax`` / ``watermark_sample``;
the top-k scheme hands over the sampler's candidate ids.  A detection service scores
batches of texts.  Batches run from one request to a thousand, vocabularies from 32000
tokens to 152064, odd sizes and vocabulary shards among them, fp32 and bf16 logits, both
seedings, windows of 1 to 8 tokens.

Each case is a dict of plain values.  Logits cases have ``B`` rows of ``V`` columns,
``dtype``, ``seeding``, ``width`` (the window) and ``offset`` (the token id of column 0, not
0 for a vocabulary shard); detection cases have ``N`` texts of up to ``L`` tokens.
"""
from __future__ import annotations

import math

import torch

import paper_2609_03844_amd as sbw

KEY = 0x243F6A8885A308D3   # a 64-bit watermark key
GAMMA = 0.25
DELTA = 2.0
INV_TEMPERATURE = 1.0 / 0.8
TEXT_VOCABULARY = 128256   # token ids of the detected texts


def _logits_case(name, op, B, V, dtype, seeding, width, offset=0, k=0):
    return dict(name=name, op=op, B=B, V=V, dtype=dtype, seeding=seeding, width=width,
                offset=offset, k=k)


def _text_case(name, N, L, seeding, width, ragged, distinct):
    return dict(name=name, op="detect", N=N, L=L, seeding=seeding, width=width, ragged=ragged,
                distinct=distinct)


def listed():
    return [
        # One interactive request on a small vocabulary: the smallest call, all latency.
        _logits_case("one_request_f32", "watermark", 1, 32000, "f32", "context", 1),
        # An ordinary serving batch whose LM head emits bf16.
        _logits_case("batch64_bf16", "watermark", 64, 128256, "bf16", "context", 1),
        # The library's headline shape: a large batch, full-vocabulary self-salt.
        _logits_case("batch256_self_salt", "watermark", 256, 152064, "f32", "self_salt", 1),
        # The paper's full-vocabulary self-salt scheme, window of four tokens.
        _logits_case("batch64_self_salt_w4", "watermark", 64, 151936, "f32", "self_salt", 4),
        # The largest batch: throughput decoding, the paper's window of four.
        _logits_case("batch1024_w4", "watermark", 1024, 152064, "f32", "context", 4),
        # A vocabulary with added tokens, so that most rows start off 16-byte alignment.
        _logits_case("odd_vocabulary", "watermark", 48, 128259, "f32", "context", 4),
        # Greedy decoding (evaluation runs) from bf16 logits.
        _logits_case("greedy_bf16", "greedy", 128, 128256, "bf16", "self_salt", 1),
        # Sampled decoding of a large batch.
        _logits_case("sample_f32", "sample", 256, 152064, "f32", "self_salt", 1),
        # The top-40 scheme: the sampler's candidates only.
        _logits_case("top40_bf16", "candidates", 256, 152064, "bf16", "self_salt", 4, k=40),
        # Corpus scan: many short texts.
        _text_case("detect_corpus", 4096, 512, "self_salt", 1, False, False),
        # A few long documents of different lengths.
        _text_case("detect_documents", 8, 16384, "context", 4, True, False),
        # Texts with repeated n-grams scored once.
        _text_case("detect_distinct", 1024, 1024, "self_salt", 4, True, True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["watermark", "watermark", "watermark", "greedy", "sample", "candidates",
                     "detect", "detect"])
    seeding = rng.choice(["context", "self_salt"])
    width = rng.choice([1, 1, 2, 3, 4, 4, 5, 8])
    if op == "detect":
        distinct = rng.random() < 0.4
        L = _log_uniform(rng, 48, 4096 if distinct else 16384)
        N = max(1, min(_log_uniform(rng, 1, 4096), (1 << 21) // L))
        c = _text_case("", N, L, seeding, width, rng.random() < 0.5, distinct)
    else:
        dtype = rng.choice(["f32", "bf16"])
        V = _log_uniform(rng, 32000, 152064)
        offset = 0
        if op != "candidates" and rng.random() < 0.3:      # one shard of 2, 4 or 8
            parts = rng.choice([2, 4, 8])
            cols = -(-V // parts)
            if rng.random() < 0.5:
                cols += -cols % 64                         # a head padded to even shards
            offset = cols * rng.randrange(1, parts)
            V = cols
        elif rng.random() < 0.5:
            V -= V % 64                                    # a padded vocabulary
        # as much work as the largest listed case does, by what bounds each path
        cells = (160 if op == "sample" else 190) * 152064
        if op in ("watermark", "greedy") and seeding == "context" and (V | offset) % 8 == 0:
            cells = 1000 * 152064
        elif width > 4 or (V | offset) % 8:
            cells = 70 * 152064
        B = max(1, min(_log_uniform(rng, 1, 1024), cells // V))
        k = rng.choice([20, 40, 50, 64, 100, 200]) if op == "candidates" else 0
        c = _logits_case("", op, B, V, dtype, seeding, width, offset, k)
    del c["name"]
    return c


# --- inputs -----------------------------------------------------------------------------

def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def ids(shape, vocabulary):
        """Token ids as texts have them, few of them frequent (log-uniform ranks)."""
        u = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
        rank = torch.exp(u * math.log(vocabulary)).to(torch.int64).clamp_(1, vocabulary) - 1
        return (rank * 48271 % vocabulary).to(torch.int32)

    if case["op"] == "detect":
        N, L, w = case["N"], case["L"], case["width"]
        tokens = ids((N, L), TEXT_VOCABULARY)
        lengths = None
        if case["ragged"]:
            low = max(w + 8, L // 2)
            lengths = torch.randint(low, L + 1, (N,), generator=g, device="cuda",
                                    dtype=torch.int32)
        if case["distinct"] and L >= 32:
            # every text repeats an early passage near its middle
            span = L // 8
            tokens[:, 3 * span:4 * span] = tokens[:, span:2 * span]
        return dict(case=case, tokens=tokens, lengths=lengths)

    B, V, offset = case["B"], case["V"], case["offset"]
    # a broad spread with a twentieth of the vocabulary raised, as next-token logits have
    logits = torch.empty((B, V), dtype=torch.float32, device="cuda").normal_(0.0, 3.0, generator=g)
    raised = torch.empty((B, V), dtype=torch.float32, device="cuda").uniform_(generator=g) < 0.05
    logits.add_(raised, alpha=8.0)
    del raised
    if case["dtype"] == "bf16":
        logits = logits.to(torch.bfloat16)
    window = ids((B, case["width"]), offset + V)
    state = dict(case=case, logits=logits, window=window[:, 0].contiguous()
                 if case["width"] == 1 else window)
    if case["op"] in ("greedy", "sample"):
        state["workspace"] = torch.empty(max(1, sbw.argmax_workspace_size(B, V)),
                                         dtype=torch.int64, device="cuda")
    if case["op"] == "sample":
        state["seeds"] = torch.randint(-(1 << 62), 1 << 62, (B,), generator=g, device="cuda",
                                       dtype=torch.int64)
    if case["op"] == "candidates":
        state["candidates"] = torch.topk(logits.float(), case["k"], dim=1).indices.to(
            torch.int32).contiguous()
    return state


def run(state):
    c = state["case"]
    if c["op"] == "detect":
        if not c["ragged"] and not c["distinct"]:
            return sbw.detect(state["tokens"], KEY, GAMMA, c["seeding"], width=c["width"])
        return sbw.detect_ex(state["tokens"], KEY, GAMMA, c["seeding"], width=c["width"],
                             lengths=state["lengths"], ignore_repeated=c["distinct"])
    if c["op"] == "watermark":
        return sbw.watermark(state["logits"], state["window"], KEY, GAMMA, DELTA, c["seeding"],
                             v_offset=c["offset"])
    if c["op"] == "candidates":
        return sbw.watermark_candidates(state["logits"], state["window"], state["candidates"],
                                        KEY, GAMMA, DELTA, c["seeding"])
    if c["op"] == "greedy":
        return sbw.watermark_argmax(state["logits"], state["window"], KEY, GAMMA, DELTA,
                                    c["seeding"], workspace=state["workspace"],
                                    v_offset=c["offset"])
    return sbw.watermark_sample(state["logits"], state["window"], KEY, GAMMA, DELTA,
                                state["seeds"], c["seeding"], INV_TEMPERATURE,
                                workspace=state["workspace"], v_offset=c["offset"])


# --- what a pass cannot do without --------------------------------------------------------

PHILOX_OPS = 58   # 32-bit operations of one Philox4x32-10 block (18 products, 40 adds and xors)


def work(case):
    w = case["width"]
    if case["op"] == "detect":
        cells = case["N"] * case["L"]
        texts = case["N"] * (12 + (4 if case["ragged"] else 0))
        return {"bytes": 4 * cells + texts, "flops": PHILOX_OPS * cells}
    B, V = case["B"], case["V"]
    size = 4 if case["dtype"] == "f32" else 2
    rows = 4 * w * B
    if case["op"] == "candidates":
        return {"bytes": B * case["k"] * (4 + 2 * size) + rows, "flops": PHILOX_OPS * B * case["k"]}
    if case["op"] == "watermark":
        # one block colours four tokens, or one token whose seed depends on it
        blocks = B * V / (4 if case["seeding"] == "context" else 1)
        return {"bytes": 2 * size * B * V + rows, "flops": PHILOX_OPS * blocks + B * V}
    # the logits read once; sampling draws the noise of every token, four a block
    blocks = B * V / 4 if case["op"] == "sample" else 0
    return {"bytes": size * B * V + rows + 8 * B, "flops": PHILOX_OPS * blocks + B * V}


def tolerance(case):
    # Colours, tokens and counts are integers.  A biased logit is one rounded addition, a
    # decoded value or score a fixed sequence of rounded operations, a z-score a fixed
    # sequence in binary64: every correct implementation gives the same bits.
    return "exact"


# --- the definitions in 64 bits -----------------------------------------------------------

_LOW = 0xFFFFFFFF


def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _mul32(a, x):
    """(high, low) words of the 64-bit product of the constant a and x, both 32-bit."""
    high = (a * (x >> 16) + ((a * (x & 0xFFFF)) >> 16)) >> 16
    return high & _LOW, (a * x) & _LOW


def _philox(counter, seed):
    """The four words of Philox4x32-10 at counter (c, 0, 0, 0) under a 64-bit key."""
    k0, k1 = seed & _LOW, (seed >> 32) & _LOW
    x0, x1 = counter, torch.zeros_like(counter)
    x2, x3 = x1, x1
    for r in range(10):
        ah, al = _mul32(0xD2511F53, x0)
        bh, bl = _mul32(0xCD9E8D57, x2)
        x0, x1 = bh ^ x1 ^ ((k0 + r * 0x9E3779B9) & _LOW), bl
        x2, x3 = ah ^ x3 ^ ((k1 + r * 0xBB67AE85) & _LOW), al
    return x0, x1, x2, x3


def _cbrng(v, seed):
    w = torch.stack(torch.broadcast_tensors(*_philox(v >> 2, seed)))
    return torch.gather(w, 0, (v & 3).expand(w.shape[1:]).unsqueeze(0))[0]


def _hash(a):
    """Jenkins' 32-bit integer hash."""
    a = (a + 0x7ED55D16 + (a << 12)) & _LOW
    a = a ^ 0xC761C23C ^ (a >> 19)
    a = (a + 0x165667B1 + (a << 5)) & _LOW
    a = ((a + 0xD3A2646C) ^ (a << 9)) & _LOW
    a = (a + 0xFD7046C5 + (a << 3)) & _LOW
    return a ^ 0xB55A4F09 ^ (a >> 16)


def _green(window, v, seeding):
    """Colour of the tokens v under windows whose last dimension is the window's."""
    key = _signed(KEY)
    if seeding == "context":
        x = _cbrng(v, key * window.sum(-1))
    else:
        flip = _signed(1 << 63)               # unsigned order of int64 values
        jv = _hash(v)
        seed = (key * jv * jv) ^ flip
        for i in range(window.shape[-1]):
            seed = torch.minimum(seed, (key * _hash(window[..., i]) * jv) ^ flip)
        x = _cbrng(v, seed ^ flip)
    return x < math.ceil(GAMMA * 2.0 ** 32)


def _detect_exact(state):
    c = state["case"]
    w, L = c["width"], c["L"]
    tokens = state["tokens"].to(torch.int64)
    N = tokens.shape[0]
    grams = tokens.unfold(1, w + 1, 1)                    # [N, L - w, w + 1]
    green = _green(grams[..., :w], grams[..., w], c["seeding"])
    lengths = (state["lengths"].to(torch.int64) if state["lengths"] is not None
               else torch.full((N,), L, device=tokens.device))
    scored = torch.arange(w, L, device=tokens.device)[None, :] < lengths[:, None]
    if c["distinct"]:
        # equal n-grams numbered alike over the batch; each text scores one of each
        text = torch.arange(N, device=tokens.device)[:, None, None].expand(N, L - w, 1)
        rows = torch.cat([text, grams], dim=2)[scored]
        unique, inverse = torch.unique(rows, dim=0, return_inverse=True)
        colour = torch.zeros(unique.shape[0], dtype=torch.int64, device=tokens.device)
        colour[inverse] = green[scored].to(torch.int64)
        T = torch.bincount(unique[:, 0], minlength=N)
        W = torch.zeros(N, dtype=torch.int64, device=tokens.device).index_add_(0, unique[:, 0], colour)
    else:
        T = scored.sum(1)
        W = (green & scored).sum(1)
    t = T.to(torch.float64)
    z = (W.to(torch.float64) - t * GAMMA) / torch.sqrt(t * GAMMA * (1.0 - GAMMA))
    W, T = W.to(torch.int32), T.to(torch.int32)
    return (W, T, z) if c["ragged"] or c["distinct"] else (W, z)


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "detect":
        return _detect_exact(s)
    window = s["window"].to(torch.int64).reshape(case["B"], case["width"])
    if case["op"] == "candidates":
        out = s["logits"].to(torch.float64)
        ids = s["candidates"].to(torch.int64)
        green = _green(window[:, None, :], ids, case["seeding"])
        return out.scatter_add_(1, ids, DELTA * green.to(torch.float64))
    v = torch.arange(case["offset"], case["offset"] + case["V"], device="cuda")
    rows = []
    for b in range(0, case["B"], 16):
        x = s["logits"][b:b + 16].to(torch.float64)
        x += DELTA * _green(window[b:b + 16, None, :], v[None, :], case["seeding"])
        if case["op"] == "sample":
            n = _cbrng(v[None, :].expand(x.shape), s["seeds"][b:b + 16, None])
            u = ((n >> 9).to(torch.float64) + 0.5) * 2.0 ** -23
            x = x * INV_TEMPERATURE - torch.log(-torch.log(u))
        # a token may be another one where two scores round alike: its score says enough
        rows.append(x if case["op"] == "watermark" else x.max(dim=1).values)
    out = torch.cat(rows)
    return out if case["op"] == "watermark" else (None, out)
