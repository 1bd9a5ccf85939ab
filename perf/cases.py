"""Performance cases of the exponent-reuse codec, through its public binding.

A case is what a sender, a receiver or both do for one tensor group in two
consecutive iterations: the weights move W -> W' and back W' -> W, so every
pass meets changed blocks, leaves the exponent caches as it found them and can
be repeated. Shapes are the workloads of ``paper_2609_04609_amd.synth``.

Keys of a case:
  mode    "step"    encode the own shard, decode the gathered shards
          "encode"  the sender alone
          "decode"  the receiver alone
          "raw"     the uncompressed form (tensors the selection rule leaves
                    out, and the first gather), encode and decode, one way
          "hashed"  the sender with the block hash in place of the cache
          "rans"    "step" with rANS-coded exceptions
  R, n    shards and values per shard; the own shard is rank R // 2's, a view
          into the flat weights
  B       block size
  fp16    fp16 values instead of bf16
  keep    how the sender's cache is brought forward: "fused" into the encode,
          by a "call" of its own, or as the own-rank "slot" of the receiver's
          caches, which the decode updates (modes step and rans)
  update  "natural" drift, "bernoulli" exponent moves at `rate`, or the same
          "clustered": 10% of the 4096-value blocks hold 90% of the moves
"""
import math

import torch

from paper_2609_04609_amd import ciera

STD = 0.02


def _case(name, mode, R, n, B, update, rate=0.0, fp16=False, keep="fused"):
    return dict(name=name, mode=mode, R=R, n=n, B=B, update=update, rate=rate,
                fp16=fp16, keep=keep)


def listed():
    olmoe, dsv3 = 25_165_824, 88_080_384  # values of one rank's layer shard
    return [
        # a layer norm of 2048 values over 16 ranks at its steady change rate:
        # the smallest tensor that a model step sends, all launches and latency
        _case("layernorm_step", "step", 16, 128, 512, "bernoulli", 0.00202),
        # one expert matrix (2048 x 1024) over 16 ranks, natural drift
        _case("expert_step", "step", 16, 131_072, 512, "natural"),
        # the tensors of one layer that the selection rule sends raw
        # (attention, router, layer norms), as one group over 16 ranks
        _case("raw_group", "raw", 16, 1_057_024, 512, "bernoulli", 0.00627),
        # a whole layer (experts, attention, router, layer norms) flattened
        # over 12 ranks: shards whose length is no multiple of 8, so that own
        # shard, caches and outputs start at odd places; caches kept once
        _case("ragged_layer_step", "step", 12, 34_963_798, 512, "bernoulli",
              0.001, keep="slot"),
        # the sender of one MoE layer at the default block size
        _case("encode_layer", "encode", 1, olmoe, 512, "bernoulli", 0.001),
        # the sender that compresses best per byte sent (B = 64) and brings
        # its cache forward in a call of its own
        _case("encode_layer_b64_call", "encode", 1, olmoe, 64, "bernoulli",
              0.001, keep="call"),
        # a fine-grained MoE layer's shard at the largest block size
        _case("encode_shard_b4096", "encode", 1, dsv3, 4096, "clustered",
              0.005),
        # the sender with the paper's hash cache
        _case("encode_layer_hashed", "hashed", 1, olmoe, 512, "bernoulli",
              0.001),
        # element-wise exceptions: both sides of one layer at B = 1
        _case("layer_step_b1", "step", 16, olmoe, 1, "bernoulli", 0.001),
        # the second precision: both sides of one layer in fp16
        _case("layer_step_fp16", "step", 16, olmoe, 512, "bernoulli", 0.001,
              fp16=True),
        # entropy-coded exceptions: both sides of one layer
        _case("layer_step_rans", "rans", 16, olmoe, 512, "bernoulli", 0.001),
        # the receiver of a fine-grained MoE layer: 16 of its ranks' shards
        _case("decode_large_layer", "decode", 16, dsv3, 512, "clustered",
              0.005),
    ]


def draw(rng):
    mode = rng.choice(["step", "step", "encode", "decode", "raw", "hashed",
                       "rans"])
    fp16 = mode in ("step", "encode", "decode", "raw") and rng.random() < 0.2
    blocks = [1, 1, 16, 32, 64, 64, 128, 256, 512, 512, 512, 1024, 2048, 4096]
    if fp16 or mode in ("hashed", "rans"):
        blocks = blocks[2:]
    B = rng.choice(blocks)
    R = rng.choice([1, 2, 3, 4, 6, 7, 8, 12, 16, 16, 16])
    # values in one shard: 64 ... 34 million, half of them multiples of 64
    n = int(math.exp(rng.uniform(math.log(64), math.log(34_000_000))))
    n = n // 64 * 64 if rng.random() < 0.5 else n | 1
    update = rng.choice(["bernoulli", "bernoulli", "natural", "clustered"])
    rate = round(math.exp(rng.uniform(math.log(1e-4), math.log(0.05))), 6)
    keep = rng.choice(["fused", "fused", "slot", "call"])
    if keep == "slot" and mode not in ("step", "rans"):
        keep = "fused"
    if mode in ("encode", "hashed"):
        R = min(R, 4)
    c = _case("", mode, R, n, B, "bernoulli" if fp16 else update,
              0.0 if update == "natural" and not fp16 else rate, fp16, keep)
    del c["name"]
    return c


def _moved(c):
    """Expected share of values whose exponent changes, and of blocks (by the
    distribution of the change rates over the 4096-value blocks)."""
    B = c["B"]
    if c["update"] == "natural":
        rates = [(1.0, 0.027)]  # measured for std 0.02, noise 1e-4
    elif c["update"] == "clustered":
        rates = [(0.1, 9.0 * c["rate"]), (0.9, c["rate"] / 9.0)]
    else:
        rates = [(1.0, c["rate"])]
    vals = sum(s * min(1.0, r) for s, r in rates)
    blks = sum(s * (1.0 - (1.0 - min(1.0, r)) ** min(B, c["n"]))
               for s, r in rates)
    return vals, blks


def work(c):
    """Bytes one pass has to move. Encode: W' and the cache (or the hashes) in,
    the encoded shard and the cache's changed bytes out. Decode: the encoded
    shards and the unchanged cache bytes in, values and changed cache bytes
    out. rANS: the coded list in place of the raw one (about 3 of 8 bits)."""
    n, R, B = c["n"], c["R"], c["B"]
    vals, blks = _moved(c)
    E = blks * n
    bm = n / B / 8
    sm, ex = (1.375 * n, 0.625 * E) if c["fp16"] else (n, E)
    wire_ex = 3 / 8 * ex if c["mode"] == "rans" else ex
    enc = 2 * n + n + sm + bm + wire_ex + 64 + vals * n
    dec = R * (sm + bm + wire_ex + 64 + (n - E) + 2 * n + E)
    if c["mode"] == "raw":
        return {"bytes": 4 * n + R * (2 * n + 2 * n + n), "flops": 0}
    if c["mode"] == "hashed":
        return {"bytes": 2 * (3 * n + bm + E + 64 + 32 * n / B), "flops": 0}
    per = {"encode": enc, "decode": dec}.get(c["mode"], enc + dec)
    return {"bytes": 2 * per, "flops": 0}


def tolerance(c):
    return "exact"  # integers and bytes: the codec is lossless


def _as_int16(w):
    return torch.where(w >= 0x8000, w - 0x10000, w).to(torch.int16)


def _exponents(bits, fp16):
    x = bits.to(torch.int32)
    return ((x >> 10) & 0x1F if fp16 else (x >> 7) & 0xFF).to(torch.uint8)


def _weights(c, seed):
    """(W, W') of all R shards, flat, as 16-bit patterns."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    total, piece = c["R"] * c["n"], 1 << 25
    W = torch.empty(total, dtype=torch.int16, device="cuda")
    W2 = torch.empty_like(W)
    top, sh = (30, 10) if c["fp16"] else (254, 7)

    def rand(k):
        return torch.rand(k, generator=g, device="cuda")

    for lo in range(0, total, piece):
        k = min(piece, total - lo)
        x = torch.randn(k, generator=g, device="cuda") * STD
        x = x.to(torch.float16 if c["fp16"] else torch.bfloat16)
        W[lo:lo + k] = x.view(torch.int16)
        if c["update"] == "natural":
            y = x.float().add_(torch.randn(k, generator=g, device="cuda"),
                               alpha=1e-4)
            W2[lo:lo + k] = y.to(torch.bfloat16).view(torch.int16)
            continue
        rate = c["rate"]
        if c["update"] == "clustered":
            hot = rand((k + 4095) // 4096) < 0.1
            rate = torch.where(hot, 9.0 * rate, rate / 9.0)
            rate = rate.repeat_interleave(4096)[:k]
        moved = rand(k) < rate
        up = rand(k) < 0.5
        b = W[lo:lo + k].to(torch.int32) & 0xFFFF
        e = (b >> sh) & ((1 << (15 - sh)) - 1)
        up = (up | (e == 0)) & (e < top)
        b = torch.where(moved, b + torch.where(up, 1 << sh, -(1 << sh)), b)
        W2[lo:lo + k] = _as_int16(b)
    return W, W2


def _gather(c, W, caches, ws):
    """The R encoded shards of W back to back and their offsets: what the
    Allgather leaves with every rank."""
    n, R, B = c["n"], c["R"], c["B"]
    bound = ciera.ciera_encoded_bound(n, B, ciera.FP16 if c["fp16"] else 0)
    buf = torch.zeros(R * bound, dtype=torch.uint8, device="cuda")
    size = torch.zeros(1, dtype=torch.int64, device="cuda")
    offs, at = [], 0
    for j in range(R):
        out = buf[at:at + bound]
        if c["mode"] == "raw":
            ciera.encode_t(W[j * n:(j + 1) * n], None, B, ws, out, raw=True,
                           out_bytes=size, fp16=c["fp16"])
        else:
            ciera.encode_t(W[j * n:(j + 1) * n], caches[j * n:(j + 1) * n], B,
                           ws, out, out_bytes=size, fp16=c["fp16"])
        if c["mode"] == "rans":
            ciera.ans_code_t(out, n, B, ws, size)
        offs.append(at)
        at += int(size.item())
    offs = torch.tensor(offs, dtype=torch.int64, device="cuda")
    return buf[:at].clone(), offs


def prepare(c, seed):
    """Weights of both iterations, caches of the first, the gathered buffers,
    workspaces and output buffers."""
    n, R, B, mode = c["n"], c["R"], c["B"], c["mode"]
    W, W2 = _weights(c, seed)
    me = R // 2
    own = slice(me * n, (me + 1) * n)
    s = dict(c, bits=(W2[own], W[own]))
    ws_dec = ciera.Workspace(n, R, B, "cuda", ans=mode == "rans")
    ws_enc = ciera.Workspace(n, 1, B, "cuda", ans=mode == "rans")
    bound = ciera.ciera_encoded_bound(n, B, ciera.FP16 if c["fp16"] else 0)
    if mode in ("encode", "hashed"):  # one shard is all the sender has
        s["send"] = _exponents(W[own], c["fp16"])
        if mode == "hashed":
            s["hash"] = torch.empty(2 * ((n + B - 1) // B), dtype=torch.int64,
                                    device="cuda")
            ciera.hash_blocks_t(W[own].contiguous(), B, s["hash"])
    else:
        cache, cache2 = _exponents(W, c["fp16"]), _exponents(W2, c["fp16"])
        gathered = [_gather(c, W2, cache, ws_dec)]
        if mode != "raw":
            gathered.append(_gather(c, W, cache2, ws_dec))
        del cache2
        s["gathered"] = gathered
        s["cache"] = cache
        s["slot"] = cache[own]
        s["send"] = s["slot"].clone()
        s["values"] = [torch.zeros_like(W) for _ in gathered]
    s["enc"] = [torch.zeros(bound, dtype=torch.uint8, device="cuda")
                for _ in range(1 if mode == "raw" else 2)]
    s.update(ws_enc=ws_enc, ws_dec=ws_dec)
    return s


def _send(s, i):
    """Encode the own shard's weights of one iteration."""
    mode, B, out = s["mode"], s["B"], s["enc"][i]
    if mode == "hashed":
        ciera.encode_hashed_t(s["bits"][i], s["hash"], s["hash"], B,
                              s["ws_enc"], out)
        return
    if mode == "raw":
        ciera.encode_t(s["bits"][i], None, B, s["ws_enc"], out, raw=True,
                       fp16=s["fp16"])
        return
    cache = s["slot"] if s["keep"] == "slot" else s["send"]
    ciera.encode_t(s["bits"][i], cache, B, s["ws_enc"], out, fp16=s["fp16"],
                   update_cache=s["keep"] == "fused")
    if s["keep"] == "call":
        ciera.update_cache_t(cache, out, s["n"], B, s["ws_enc"],
                             fp16=s["fp16"])
    if mode == "rans":
        ciera.ans_code_t(out, s["n"], B, s["ws_enc"])


def _receive(s, i):
    """Decode what the Allgather of one iteration left."""
    gathered, offsets = s["gathered"][i]
    ciera.decode_gathered_t(gathered, offsets, s["n"], s["B"], s["values"][i],
                            s["cache"], s["ws_dec"], fp16=s["fp16"])


def run(s):
    """Both iterations (raw: one): W -> W' and W' -> W."""
    for i in range(len(s["enc"])):
        if s["mode"] != "decode":
            _send(s, i)
        if s["mode"] not in ("encode", "hashed"):
            _receive(s, i)
    out = {}
    if s["mode"] != "decode":
        out["encoded"] = s["enc"]  # the encoded bytes, then zeros or leftovers
        if s["mode"] == "hashed":
            out["hash"] = s["hash"]
        elif s["keep"] != "slot" and s["mode"] != "raw":
            out["send"] = s["send"]
    if s["mode"] not in ("encode", "hashed"):
        out["values"], out["cache"] = s["values"], s["cache"]
    return out


def exact(c, seed):
    """Values and caches by plain integer arithmetic; the encoded bytes have no
    form other than the codec's own."""
    me, n, mode = c["R"] // 2, c["n"], c["mode"]
    if mode == "hashed":
        return None
    W, W2 = _weights(c, seed)
    own = W[me * n:(me + 1) * n]
    # after W -> W' -> W the caches hold W's exponents again
    out = {}
    if mode != "decode":
        out["encoded"] = None
        if c["keep"] != "slot" and mode != "raw":
            out["send"] = _exponents(own, c["fp16"])
    if mode != "encode":
        out["values"] = [W2] if mode == "raw" else [W2, W]
        out["cache"] = _exponents(W2 if mode == "raw" else W, c["fp16"])
    return out
