"""Performance cases of the activation codec: what a pipeline stage has it do, through the package's public calls.

A case is a plain dict:
  kind     "encode"   activations -> stream                            (the sending stage)
           "decode"   stream -> activations                            (the receiving stage)
           "trip"     both, one after the other                        (what bench.py calls a step)
           "samples"  sample by sample, each stream decoded on arrival (encode overlapped with send)
           "grad"     the fixed-point compressor of the backward pass, there and back
  dtype    "bf16" or "f32": storage type of the tensor; "out": type the decoder writes
  batch, seq, hidden   the contiguous tensor [batch, seq, hidden]
  tile, alloc_tile, scope, low_bits, budget   fields of tahq_config (include/tahq.h)
  bits, scale          fields of tahq_naive_config ("grad" only)
  recipe   distribution of the tensor, see _tensor()
"""
import math

import torch

import paper_2506_01352_amd as tahq

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_TAHQ = {"f32": tahq.F32, "bf16": tahq.BF16}


def _case(kind, dtype, batch, seq, hidden, tile=64, budget=3.8, recipe="tokens", **more):
    c = {"kind": kind, "dtype": dtype, "out": dtype, "batch": batch, "seq": seq, "hidden": hidden, "recipe": recipe}
    if kind == "grad":
        c.update({"bits": 8, "scale": 16384.0})
    else:
        c.update({"tile": tile, "alloc_tile": 0, "scope": 0, "low_bits": 3, "budget": budget})
    c.update(more)
    return c


def _named(name, c):
    c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a toy stage's boundary (128 tokens x 512 channels), one width for all tiles.  Host and launch
        # latency are all of it.
        _named("trip_f32_1x128x512_b4.0", _case("trip", "f32", 1, 128, 512, 64, 4.0, "channels")),
        # One sample of the micro-batch a small GPT-style model is trained with (1024 tokens x 1600 channels) at the usual
        # mean width of 3.8 bits: the sending stage of a pipeline with micro-batch 1.
        _named("encode_bf16_1x1024x1600_b3.8", _case("encode", "bf16", 1, 1024, 1600)),
        # The receiving stage of the same model with two samples per micro-batch.
        _named("decode_bf16_2x1024x1600_b3.8", _case("decode", "bf16", 2, 1024, 1600)),
        # fp32 activations of a small model, half of the tiles wide: both directions.
        _named("trip_f32_4x512x2048_b3.5", _case("trip", "f32", 4, 512, 2048, 64, 3.5, "lognormal")),
        # Tiles of 128 channels, every tile 3 bits wide: single-pass encode, heavy-tailed values.
        _named("trip_bf16_8x1024x4096_g128_b3.0", _case("trip", "bf16", 8, 1024, 4096, 128, 3.0, "heavy")),
        # The configuration the headline metric is quoted on, sending and receiving side.
        _named("encode_bf16_8x4096x8192_b3.25", _case("encode", "bf16", 8, 4096, 8192, 64, 3.25)),
        _named("decode_bf16_8x4096x8192_b3.25", _case("decode", "bf16", 8, 4096, 8192, 64, 3.25)),
        # Tiles of 32 channels, 4 bits throughout, sparse values and dead tokens.
        _named("trip_bf16_16x2048x5120_g32_b4.0", _case("trip", "bf16", 16, 2048, 5120, 32, 4.0, "sparse")),
        # Token-level allocation: every token's channels share one width, tokens are ranked.
        _named("encode_bf16_4x2048x4096_token_b3.8", _case("encode", "bf16", 4, 2048, 4096, alloc_tile=4096)),
        # An odd sequence length and small tiles with the INT2/INT3 mix: ranking units that are no multiple of anything.
        _named("trip_bf16_3x777x1600_g16_b2.25", _case("trip", "bf16", 3, 777, 1600, 16, 2.25, low_bits=2)),
        # Sample-wise use in a pipeline: eight samples, each a stream of its own that is decoded when it is there.
        _named("samples_bf16_8x1024x1600_b3.8", _case("samples", "bf16", 8, 1024, 1600)),
        # The backward direction: 8-bit fixed-point codes of rescaled activation gradients.
        _named("grad_bf16_16x2048x5120_8bit", _case("grad", "bf16", 16, 2048, 5120, recipe="sparse")),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, 64 K to 128 M elements, all tile widths, even and odd lengths, the options in use."""
    kind = rng.choice(["encode", "encode", "encode", "decode", "decode", "trip", "trip", "samples", "grad"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    tile = rng.choice([8, 16, 32, 32, 64, 64, 64, 64, 128])
    hidden = rng.choice([512, 768, 1024, 1600, 2048, 2560, 3072, 4096, 5120, 8192])
    if tile == 128 and hidden % 128:
        hidden = 1536
    # narrow tiles and fp32 cost more per element: their sizes end earlier
    top = 1 << (27 - (1 if dtype == "f32" else 0) - (1 if tile < 32 else 0) - (1 if kind in ("trip", "samples") else 0))
    elements = _log_uniform(rng, 1 << 16, top)
    batch = rng.randint(2, 8) if kind == "samples" else min(rng.choice([1, 1, 2, 3, 4, 8, 16]), max(1, elements // (32 * hidden)))
    seq = max(16, elements // (batch * hidden))
    if seq >= 64 and rng.random() < 0.5:
        seq -= seq % 64                              # as often as not a round length
    recipe = rng.choice(["tokens", "tokens", "channels", "lognormal", "heavy", "sparse"])
    if kind == "grad":
        return _case(kind, dtype, batch, seq, hidden, recipe="sparse", bits=rng.choice([4, 6, 8, 8, 10]),
                     scale=float(1 << rng.randint(10, 16)))
    low = rng.choice([3, 3, 3, 3, 2])
    budget = low + rng.choice([0.0, 0.25, 0.5, 0.8, 0.8, 0.8, 1.0, round(rng.uniform(0.05, 0.95), 2)])
    c = _case(kind, dtype, batch, seq, hidden, tile, budget, recipe, low_bits=low)
    if rng.random() < 0.2:
        c["alloc_tile"] = rng.choice([hidden, hidden, 2 * tile if hidden % (2 * tile) == 0 else hidden])
    if kind != "samples" and rng.random() < 0.15:
        c["scope"] = 1
    if kind == "decode" and rng.random() < 0.25:
        c["out"] = "f32"
    return c


def _tensor(case, seed):
    """Stand-in for a boundary tensor, made on the GPU: the distributions of the repository's synthetic workloads.
      tokens     N(0,1), one token in twenty U[-8,8] instead; a few channels x40
      channels   N(0,1); a few channels x20
      lognormal  N(0,1), one channel in a hundred x10..50, tokens scaled by LogNormal(0, 0.5)
      heavy      Student-t with 3 degrees of freedom; a few channels x30
      sparse     N(0, 1e-3), one element in a thousand x1000, one token in five all zero"""
    B, S, C = case["batch"], case["seq"], case["hidden"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dev = {"device": "cuda", "generator": g}
    recipe = case["recipe"]
    few = torch.randperm(C, **dev)[:max(1, C // 256)]
    hundredth = torch.randperm(C, **dev)[:max(1, C // 100)]
    gain = torch.empty(hundredth.numel(), device="cuda").uniform_(10.0, 50.0, generator=g)
    out = torch.empty(B, S, C, dtype=_TORCH[case["dtype"]], device="cuda")
    for b in range(B):
        x = torch.randn(S, C, **dev)
        if recipe == "tokens":
            wide = torch.rand(S, 1, **dev) < 0.05
            x = torch.where(wide, torch.empty_like(x).uniform_(-8.0, 8.0, generator=g), x)
            x[:, few] *= 40.0
        elif recipe == "channels":
            x[:, few] *= 20.0
        elif recipe == "lognormal":
            x[:, hundredth] *= gain
            x *= torch.exp(0.5 * torch.randn(S, 1, **dev))
        elif recipe == "heavy":
            chi2 = torch.zeros_like(x)
            for _ in range(3):
                chi2 += torch.randn(S, C, **dev) ** 2
            x /= torch.sqrt(chi2 / 3.0)
            x[:, few] *= 30.0
        else:
            x *= torch.where(torch.rand(S, C, **dev) < 1e-3, 1.0, 1e-3)
            x *= (torch.rand(S, 1, **dev) >= 0.2)
        out[b] = x
    return out


def _config(case):
    return tahq.make_config(case["batch"], case["seq"], case["hidden"], case["tile"], _TAHQ[case["dtype"]], case["budget"],
                            scope=case["scope"], alloc_tile=case["alloc_tile"], low_bits=case["low_bits"])


def prepare(case, seed):
    kind = case["kind"]
    x = _tensor(case, seed)
    state = {"case": case, "x": x}
    if kind == "grad":
        cfg = tahq.make_naive_config(case["batch"], case["seq"], case["hidden"], _TAHQ[case["dtype"]], case["bits"],
                                     case["scale"])
        state["cfg"] = cfg
        state["packed"] = torch.empty(tahq.tahq_naive_packed_size(cfg), dtype=torch.uint8, device="cuda")
        state["out"] = torch.empty(x.numel(), dtype=_TORCH[case["out"]], device="cuda")
        return state
    cfg = _config(case)
    if kind == "samples":
        n, size, scratch = case["batch"], tahq.tahq_samples_packed_size(cfg, 1), tahq.tahq_samples_workspace_size(cfg, 1)
        state["cfg"] = cfg
        state["packed"] = [torch.empty(size, dtype=torch.uint8, device="cuda") for _ in range(n)]
        state["workspace"] = torch.empty(scratch, dtype=torch.uint8, device="cuda")
        state["out"] = torch.empty(x.numel(), dtype=_TORCH[case["out"]], device="cuda")
        return state
    codec = tahq.Codec(cfg, device="cuda", out_dtype=_TAHQ[case["out"]])
    state["codec"] = codec
    if kind == "decode":
        codec.encode(x)              # what the sending stage has sent; the receiver does not have the tensor
        del state["x"]
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "encode":
        return state["codec"].encode(state["x"])
    if kind == "decode":
        return state["codec"].decode()
    if kind == "trip":
        packed = state["codec"].encode(state["x"])
        return packed, state["codec"].decode()
    cfg, x, out = state["cfg"], state["x"], state["out"]
    if kind == "samples":
        dtype = _TAHQ[case["out"]]
        for i, packed in enumerate(state["packed"]):
            tahq.tahq_encode_samples(cfg, i, 1, x, packed, state["workspace"])
            tahq.tahq_decode_samples(cfg, i, 1, packed, out, dtype)
        return state["packed"], out
    tahq.tahq_naive_encode(cfg, x, state["packed"])
    tahq.tahq_naive_decode(cfg, state["packed"], out, _TAHQ[case["out"]])
    return state["packed"], out


def work(case):
    """Bytes: the tensor and the stream, each once per direction.  Operations per element: Eq. 1-2 (magnitude, norm, product,
    logarithm, product, sum) where tiles are ranked, the two largest magnitudes, the range and the affine code on the
    sending side; the affine map on the receiving side."""
    kind = case["kind"]
    n = case["batch"] * case["seq"] * case["hidden"]
    size = {"f32": 4, "bf16": 2}
    if kind == "grad":
        packed = tahq.tahq_naive_packed_size(tahq.make_naive_config(case["batch"], case["seq"], case["hidden"],
                                                                    _TAHQ[case["dtype"]], case["bits"], case["scale"]))
        return {"bytes": n * (size[case["dtype"]] + size[case["out"]]) + 2 * packed, "flops": 5 * n}
    cfg = _config(case)
    if kind == "samples":
        packed = case["batch"] * tahq.tahq_samples_packed_size(cfg, 1)
    else:
        packed = tahq.tahq_packed_size(cfg)
    ranked = 0.0 < case["budget"] - case["low_bits"] < 1.0
    send = {"bytes": n * size[case["dtype"]] + packed, "flops": n * (13 if ranked else 7)}
    receive = {"bytes": packed + n * size[case["out"]], "flops": n * 2}
    if kind == "encode":
        return send
    if kind == "decode":
        return receive
    return {k: send[k] + receive[k] for k in send}


def tolerance(case):
    # the stream is bytes, the decoded values follow from them by a fixed order of fp32 operations
    return "exact"
