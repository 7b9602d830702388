"""The work that users of the codec have it do, as cases that can be timed.

A case is a dict of plain values:

  op      "decode" or "encode" (one tensor), "decode_batch" or "encode_batch"
          (a checkpoint's tensors through one prepared hipGraph),
          "compress_batch" (the same encode without preparation), "serve"
  dtype   "bf16", "fp16", "fp32" or "fp8"
  values  what the tensor holds: "normal" (a projection), "norm" (a norm
          vector, 1 + N(0, 0.05)), "rows" (rows of differing spread) or
          "pruned" (a share of the weights set to zero)
  n       elements of a single tensor; rows, cols of a "rows" matrix
  layers, hidden, kv, ffn, vocab   the checkpoint of a batch
  delta   the tensors are a fine-tuned copy, stored as the XOR delta
  chunk, S, g, exponent, policy    format parameters (0 and "" take the
          defaults)
  header  decode with a host copy of the container's header, queued without
          a host round trip; else the plain blocking call
  requests, max_bytes, mix   a burst of serving requests of log-uniform size
          (mix: the seed of their sizes and types)

`listed` gives the cases, `draw` more of the same ranges.  Inputs come from
the package's seeded generators; the codec is lossless, so every output is
bytes or words that must come back exactly.
"""
from __future__ import annotations

import math

import torch

from paper_2411_05239_amd import workloads
from paper_2411_05239_amd import zipnn as Z

WIDTH = {"bf16": 2, "fp16": 2, "fp32": 4, "fp8": 1}
CODE = {"bf16": Z.ZIPNN_BF16, "fp16": Z.ZIPNN_FP16, "fp32": Z.ZIPNN_FP32, "fp8": Z.ZIPNN_FP8_E4M3}
TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32, "fp8": torch.float8_e4m3fn}
# container bytes per input byte: closed-form entropies of the generators'
# distributions at the default parameters (deltas: see `_ratio`)
RATIO = {"bf16": 0.674, "fp16": 0.847, "fp32": 0.859, "fp8": 0.81}

_codec = None


def _shared_codec() -> "Z.Codec":
    """A program keeps one codec for its GPU."""
    global _codec
    if _codec is None:
        _codec = Z.Codec(torch.cuda.current_device())
    return _codec


def _case(op: str, name: str = "", **kw) -> dict:
    c = {"op": op, "dtype": "bf16", "values": "normal", "delta": False, "chunk": 0, "S": 0, "g": 0,
         "exponent": False, "policy": ""}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed() -> list[dict]:
    return [
        # the smallest call: one RMSNorm vector of an 8B decoder restored by the
        # plain blocking call (host and launch latency, one work item)
        _case("decode", "decode_norm_vector", values="norm", n=4096),
        # one 8 MiB projection shard restored by a loader that kept the headers:
        # few work items, the serial length of a sub-stream counts
        _case("decode", "decode_bf16_8mb", n=4_194_304, policy="huf,raw", header=True),
        # a serving corpus FP8 tensor of a ragged length (one byte group)
        _case("decode", "decode_fp8_ragged", dtype="fp8", n=37_748_753, header=True),
        # a 256 MiB FP32 matrix, two of its four byte groups coded
        _case("decode", "decode_fp32_256mb", dtype="fp32", values="rows", rows=8192, cols=8192, header=True),
        # loading one file of a sharded 8B checkpoint (about 5 GB: the embedding
        # and nine layers, 82 tensors), batched at the autotuner's usual pick
        _case("decode_batch", "decode_shard_5gb", layers=9, hidden=4096, kv=1024, ffn=14336, vocab=128256,
              chunk=262144, S=512),
        # a fine-tuned copy restored from its XOR delta and the resident base
        # (zero-aware coding), at the shape the autotuner picks for deltas
        _case("decode_batch", "decode_delta", layers=4, hidden=4096, kv=1024, ffn=14336, vocab=0, delta=True,
              chunk=1048576, S=2048),
        # a burst of requests of mixed types and sizes to the resident server
        _case("serve", "serve_burst", requests=48, max_bytes=64 << 20, mix=3000),
        # compressing the smallest tensor of a checkpoint on its own
        _case("encode", "encode_norm_vector", values="norm", n=4096),
        # compressing one 8 MiB BF16 tensor
        _case("encode", "encode_bf16_8mb", n=4_194_304, policy="huf,raw"),
        # compressing a 256 MiB FP32 matrix, every byte group tried
        _case("encode", "encode_fp32_256mb", dtype="fp32", values="rows", rows=8192, cols=8192),
        # saving the same 5 GB file again and again with a prepared encoder
        _case("encode_batch", "encode_shard_5gb", layers=9, hidden=4096, kv=1024, ffn=14336, vocab=128256,
              chunk=262144, S=512),
        # storing a fine-tuned copy as a delta (default parameters, one call)
        _case("compress_batch", "compress_delta", layers=4, hidden=4096, kv=1024, ffn=14336, vocab=0, delta=True),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    op = rng.choice(["decode", "encode", "decode", "encode", "decode_batch", "encode_batch", "compress_batch", "serve"])
    if op == "serve":
        return _case(op, requests=rng.randint(8, 64), max_bytes=_log_int(rng, 1 << 20, 64 << 20),
                     mix=rng.randint(0, 1 << 20))
    if op in ("decode", "encode"):
        dtype = rng.choice(["bf16", "bf16", "fp16", "fp32", "fp8"])
        n = _log_int(rng, 4096, 268_435_456) // WIDTH[dtype]
        c = _case(op, dtype=dtype, n=max(1, n), values=rng.choice(["normal", "normal", "norm", "pruned"]),
                  delta=rng.random() < 0.2, exponent=dtype in ("bf16", "fp32") and rng.random() < 0.2)
        if dtype == "fp8":
            c.update(values="normal", delta=False)
        if op == "decode":
            c["header"] = rng.random() < 0.6
    else:
        hidden = rng.choice([512, 1024, 2048, 4096])
        c = _case(op, layers=rng.randint(1, 6), hidden=hidden, kv=hidden // 4, ffn=hidden * 7 // 2,
                  vocab=rng.choice([0, 0, 32000]) + rng.randint(0, 1), delta=rng.random() < 0.4)
    if rng.random() < 0.6:
        w = WIDTH[c["dtype"]]
        c["chunk"] = rng.choice([65536, 131072, 262144, 524288, 1048576])
        c["S"] = min(4096, c["chunk"] // w // rng.choice([128, 256, 256, 512]))
        c["g"] = rng.choice([2, 4, 4, 8])
    return c


# ------------------------------------------------------------------ inputs

def _params(case: dict) -> "Z.zipnn_params":
    names = {"auto": Z.ZIPNN_AUTO, "huf": Z.ZIPNN_HUF, "raw": Z.ZIPNN_RAW, "zg": Z.ZIPNN_ZG}
    policy = [names[t] for t in case["policy"].split(",")] if case["policy"] else None
    return Z.make_params(CODE[case["dtype"]], chunk_bytes=case["chunk"] or None, S=case["S"] or None,
                         g=case["g"] or None, policy=policy, exponent=case["exponent"] or None)


def _one(case: dict, seed: int):
    """-> (tensor, XOR base or None), on the GPU"""
    dev, dtype, values = "cuda", case["dtype"], case["values"]
    if values == "rows":
        x = workloads.fp32_rows(case["rows"], case["cols"], seed=seed, device=dev).reshape(-1).to(TORCH[dtype])
    elif dtype == "fp8":
        x = workloads.make_corpus_tensor(workloads.CorpusItem(0, "fp8", case["n"], seed), device=dev)
    else:
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        x = torch.randn(case["n"], generator=g, device=dev) * (0.05 if values == "norm" else 0.02)
        x = (x + 1.0 if values == "norm" else x).to(TORCH[dtype])
        if values == "pruned":
            x = workloads.pruned(x, 0.25, seed + 1)
    if not case["delta"]:
        return x, None
    # the fine-tuned copy keeps the word type of its base
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 2)
    hit = torch.rand(x.numel(), generator=g, device=dev) < 0.1
    z = torch.randn(x.numel(), generator=g, device=dev) * 1e-4
    return (x.float() + hit * z).to(x.dtype), x


def _checkpoint(case: dict, seed: int):
    """-> (tensors, bases or None): the tensors of a decoder checkpoint without
    the output head, so that vocab = 0 leaves the layers alone"""
    specs = workloads.checkpoint_8b_specs(case["layers"], case["hidden"], case["kv"], case["ffn"],
                                          max(1, case["vocab"]), seed0=1000 * (seed + 1))
    keep = [s for s in specs[:-1] if s.name != "embed" or case["vocab"]]
    base = [workloads.make_tensor(s, device="cuda") for s in keep]
    if not case["delta"]:
        return base, None
    return [workloads.finetune_delta(w, seed=s.seed + 7) for w, s in zip(base, keep)], base


def _corpus(case: dict, seed: int):
    items = workloads.serving_corpus(case["requests"], seed=case["mix"], max_bytes=case["max_bytes"])
    return [workloads.make_corpus_tensor(workloads.CorpusItem(it.index, it.dtype, it.nbytes, 1000 * seed + it.index),
                                         device="cuda") for it in items]


def _arena(xs, p):
    """The buffer that a program keeps for containers, large enough for any
    data (cleared, so that what lies past the containers is the same for all)."""
    cap = sum(Z.zipnn_compress_bound(Z.torch_dtype_code(x.dtype), x.numel(), p) + 127 for x in xs)
    return torch.zeros(cap, dtype=torch.uint8, device="cuda")


def _flat_outputs(xs):
    """One allocation for all outputs (a loader's weight buffer), each at a
    256-byte aligned offset: -> (words of the whole buffer, the views)."""
    offs, end = [], 0
    for x in xs:
        offs.append(end)
        end += (x.numel() * x.element_size() + 255) // 256 * 256
    flat = torch.zeros(end, dtype=torch.uint8, device="cuda")
    views = [flat[o:o + x.numel() * x.element_size()].view(x.dtype) for o, x in zip(offs, xs)]
    return flat.view(torch.int16), views


_BITS = {1: torch.uint8, 2: torch.int16, 4: torch.int32}


def _bits(x):
    """A tensor's words as whole numbers."""
    return x.view(_BITS[x.element_size()])


# ------------------------------------------------------------------ one pass

def prepare(case: dict, seed: int) -> dict:
    codec, op = _shared_codec(), case["op"]
    st = {"op": op, "codec": codec}
    if op == "serve":
        xs = _corpus(case, seed)
        cs = [codec.compress(x).clone() for x in xs]
        pool = sum(x.numel() * x.element_size() + 256 for x in xs) + (1 << 20)
        st["server"] = Z.Server(codec, pool, max_inflight=len(xs))
        st["handles"] = [st["server"].register(c) for c in cs]
        st["held"] = []
        return st
    p = st["params"] = _params(case)
    if op in ("decode", "encode"):
        x, base = _one(case, seed)
        st["base"] = base
        if op == "encode":
            st["x"], st["arena"] = x, _arena([x], p)
        else:
            st["container"] = codec.compress(x, p, base=base).clone()
            st["out"] = torch.empty_like(x)
            st["header"] = st["container"][:64].cpu().numpy().tobytes() if case.get("header") else None
        return st
    xs, bases = _checkpoint(case, seed)
    if op == "decode_batch":
        arena, offs = codec.compress_batch(xs, p, bases=bases)
        arena = arena[: offs[-1]].clone()
        st["flat"], outs = _flat_outputs(xs)
        st["batch"] = codec.prepare_batch(arena, offs, outs, bases)
    elif op == "encode_batch":
        st["encoder"] = codec.prepare_encoder(xs, p, bases, arena=_arena(xs, p))
    else:
        st["xs"], st["bases"], st["arena"] = xs, bases, _arena(xs, p)
    return st


def run(st: dict):
    codec, op = st["codec"], st["op"]
    if op == "decode":
        # with the header in hand the decode is only queued; the plain call
        # waits for it and checks the status
        codec.decompress(st["container"], st["out"], base=st["base"], header=st["header"],
                         check=st["header"] is None)
        return _bits(st["out"])
    if op == "encode":
        c = codec.compress(st["x"], st["params"], base=st["base"], out=st["arena"])
        return st["arena"], c.numel()
    if op == "decode_batch":
        st["batch"].run()
        return st["flat"]
    if op == "encode_batch":
        offs = st["encoder"].run()
        return st["encoder"].arena, torch.tensor(offs)
    if op == "compress_batch":
        arena, offs = codec.compress_batch(st["xs"], st["params"], bases=st["bases"], arena=st["arena"])
        return arena, torch.tensor(offs)
    # a burst: the last burst's outputs are given back, then every container
    # is asked for once and the results are used where they lie in the pool
    srv = st["server"]
    for t in st["held"]:
        srv.release(t)
    tickets = [srv.submit(h) for h in st["handles"]]
    done = 0
    while done < len(tickets):
        if srv.next_done() is not None:
            done += 1
    st["held"] = tickets
    outs = [srv.output(t, h) for t, h in zip(tickets, st["handles"])]
    for o in outs:
        o.server = srv   # the outputs lie in the server's pool: they keep it alive
    return outs


# ------------------------------------------------------------------ its cost

def _ratio(case: dict) -> float:
    if case["delta"]:
        return 0.075 if case["dtype"] == "bf16" else 0.2
    if case["values"] == "pruned":
        return 0.3
    return RATIO[case["dtype"]]


def _elements(case: dict) -> int:
    if case["op"] in ("decode", "encode"):
        return case["rows"] * case["cols"] if case["values"] == "rows" else case["n"]
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return case["layers"] * (2 * h * h + 2 * kv * h + 3 * f * h + 2 * h) + h + case["vocab"] * h


def work(case: dict) -> dict:
    """Each direction reads one side (and the XOR base) and writes the other."""
    if case["op"] == "serve":
        # sizes are log-uniform from 64 KiB: the mean of that distribution
        lo, hi = 65536, case["max_bytes"]
        u = case["requests"] * (hi - lo) / math.log(hi / lo)
        return {"bytes": u * (1 + 0.75), "flops": 0}
    u = _elements(case) * WIDTH[case["dtype"]]
    return {"bytes": u * (1 + _ratio(case) + (1 if case["delta"] else 0)), "flops": 0}


def exact(case: dict, seed: int):
    """The codec is lossless: a decode returns the words that were stored.
    Containers have no value in plain arithmetic."""
    if case["op"] == "decode":
        return _bits(_one(case, seed)[0])
    return None
