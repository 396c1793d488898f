"""The capture-and-stage work whose speed matters to a user, as cases that can be timed and compared.

Four kinds of case, one per way in which a program reaches the library:

  into     dmi_observe_into: one dense tensor, the record written into the caller's device memory
  step     one decode step through a ring: every observation point of the step captured (one call
           per point as the hooks fire, or one batched call), drained to the pinned host ring and polled
  kv       the same for K and V slices of several layers of a paged cache
  replay   a step of HookPoints captured once in a graph and replayed, then drained and polled

Ring cases end with dmi_drain(FLUSH) and dmi_poll_host: the pass is over when its records can be read
on the host.  Outputs are whole records, split by section (header and request table, payload,
one array per summary; pads are part of the section in front of them); sequence numbers are given
relative to the pass's first one, because a ring goes on counting.
"""
import ctypes
import gc
import math
import random

import numpy as np
import torch

from paper_2605_11093_amd import binding as B
from paper_2605_11093_amd import hookpoint as H

DEV = "cuda:0"
STEP_ID = 7
TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
CODE = {"none": B.DT_NONE, "bf16": B.DT_BF16, "fp16": B.DT_FP16, "fp32": B.DT_FP32, "fp8": B.DT_FP8}
SIZE = {"none": 0, "fp8": 1, "bf16": 2, "fp16": 2, "fp32": 4}
SUMS = (("l2", B.SUM_L2), ("mean", B.SUM_MEAN), ("absmax", B.SUM_ABSMAX))


def _into(name, dtype, width, reqs, sel, out, sums, **more):
    return {"name": name, "kind": "into", "dtype": dtype, "width": width, "reqs": reqs, "sel": sel, "out": out,
            "sums": sums, "len_lo": 0, "len_hi": 0, "every": 1, "lead": 0, "keep": False, **more}


def _kv(name, layers, reqs, ctx_lo, ctx_hi, out, sums, **more):
    return {"name": name, "kind": "kv", "dtype": "bf16", "layers": layers, "reqs": reqs, "seqs": 128, "ctx_lo": ctx_lo,
            "ctx_hi": ctx_hi, "block": 16, "heads": 8, "take": 2, "dim": 128, "out": out, "sums": sums, **more}


def listed():
    return [
        # the last token of four short requests, as in the smallest configuration: nothing but latency
        _into("into_tiny", "bf16", 256, 4, "last", "bf16", 0),
        # one layer's residual stream at a decode step of an 8B-shaped model, with norms for monitoring
        _into("into_decode_stats", "bf16", 4096, 64, "last", "bf16", B.SUM_L2 | B.SUM_ABSMAX),
        # ragged prompts, every fourth token of the residual stream, stored as fp8
        _into("into_prefill_fp8", "bf16", 4096, 32, "ragged", "fp8", 0, len_lo=128, len_hi=2048, every=4),
        # the same prompts at the MLP's intermediate width: the largest single record
        _into("into_prefill_mlp_fp8", "bf16", 14336, 32, "ragged", "fp8", 0, len_lo=128, len_hi=2048, every=4),
        # logits of a decode batch over a vocabulary of odd size: rows that no 16-byte grid fits
        _into("into_logits_odd", "bf16", 50257, 64, "last", "bf16", 0),
        # per-token statistics only of a hidden state kept in fp32, half of the requests kept (best effort)
        _into("into_prefill_stats_keep", "fp32", 4096, 16, "ragged", "none", 7, len_lo=128, len_hi=2048, keep=True),
        # the smallest configuration's step: eight hooks, one call each, records read on the host
        {"name": "step_tiny", "kind": "step", "dtype": "bf16", "points": 8, "reqs": 4, "width": 256, "batch": False,
         "out": "bf16", "sums": 0},
        # an 8B-shaped decode step: all 32 layers in one launch, raw rows and norms, delivered
        {"name": "step_decode", "kind": "step", "dtype": "bf16", "points": 32, "reqs": 64, "width": 4096, "batch": True,
         "out": "bf16", "sums": B.SUM_L2 | B.SUM_ABSMAX},
        # a 70B-shaped decode step of 256 requests at all 80 layers, of which only the statistics leave the GPU
        {"name": "step_wide_stats", "kind": "step", "dtype": "bf16", "points": 80, "reqs": 256, "width": 8192,
         "batch": True, "out": "none", "sums": 7},
        # K and V of four layers, two of eight heads, whole contexts of sixteen requests, delivered raw
        _kv("kv_raw", 4, 16, 512, 8192, "bf16", 0),
        # the same rows, only their norms and largest magnitudes
        _kv("kv_stats", 4, 16, 512, 8192, "none", B.SUM_L2 | B.SUM_ABSMAX),
        # a graph-captured step with a HookPoint behind each of 32 layers, stored as fp8
        {"name": "replay_hooks_fp8", "kind": "replay", "dtype": "bf16", "points": 32, "reqs": 64, "width": 4096,
         "out": "fp8", "sums": 0},
    ]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A row length: mostly a multiple of 64 as models have them, sometimes any number."""
    w = _log(rng, lo, hi)
    return w if rng.random() < 0.25 else max(64, w // 64 * 64)


def _types(rng):
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp16", "fp32"])
    out = rng.choice([dtype, dtype, "fp8", "fp16", "none"] if dtype == "bf16" else [dtype, dtype, "none"])
    sums = rng.choice([0, 0, B.SUM_ABSMAX, B.SUM_L2 | B.SUM_ABSMAX, 7])
    if out == "none" and not sums:
        sums = B.SUM_L2
    return dtype, out, sums


def draw(rng):
    kind = rng.choice(["into"] * 5 + ["step", "step", "kv", "kv", "replay"])
    dtype, out, sums = _types(rng)
    if kind == "into":
        sel = rng.choice(["last", "slots", "ragged", "ragged", "index"])
        if sel in ("last", "slots"):
            reqs, width, lo, hi = _log(rng, 1, 512), _width(rng, 64, 65536), 0, 0
        else:
            reqs, width = _log(rng, 1, 64), _width(rng, 64, 16384)
            hi = _log(rng, 16, 2048)
            lo = rng.randint(1, hi)
        c = _into("", dtype, width, reqs, sel, out, sums, len_lo=lo, len_hi=hi,
                  every=rng.choice([1, 1, 4]) if sel == "ragged" else 1,
                  lead=rng.choice([0, 0, 0, rng.randint(1, 64)]), keep=rng.random() < 0.25)
    elif kind == "step":
        c = {"kind": kind, "dtype": dtype, "points": _log(rng, 2, 96), "reqs": _log(rng, 1, 256),
             "width": _width(rng, 256, 8192), "batch": rng.random() < 0.7, "out": out, "sums": sums}
    elif kind == "kv":
        dtype = "fp16" if dtype == "fp32" else dtype
        out = rng.choice([dtype, "none"])
        heads = rng.choice([2, 4, 8, 16])
        hi = _log(rng, 64, 8192)
        c = _kv("", rng.randint(1, 4), _log(rng, 1, 32), rng.randint(1, hi), hi, out, sums or B.SUM_L2, dtype=dtype,
                seqs=32, block=rng.choice([16, 16, 32, 64]), heads=heads, take=rng.randint(1, min(heads, 8)),
                dim=rng.choice([64, 80, 96, 128, 128, 256]))
        if c["out"] != "none":
            c["sums"] = sums
    else:
        c = {"kind": kind, "dtype": dtype, "points": _log(rng, 2, 64), "reqs": _log(rng, 1, 256),
             "width": _width(rng, 256, 8192), "out": out, "sums": sums}
    c.pop("name", None)
    # no dearer than the listed ones: bytes read, and bytes over the host link
    while True:
        n, record, read, records = _geometry(c)
        if read * records <= 600 << 20 and (kind == "into" or record * records <= 256 << 20):
            return c
        for k in ("points", "layers", "reqs", "ctx_hi", "len_hi", "width"):
            if c.get(k, 0) > 1 and rng.random() < 0.5:
                c[k] = max(1, c[k] // 2)
        for lo, hi in (("ctx_lo", "ctx_hi"), ("len_lo", "len_hi")):
            if lo in c:
                c[lo] = min(c[lo], c[hi])


# ------------------------------------------------------------------ what a case asks for
def _lengths(c):
    """(tokens, kept) per request: the case alone fixes them, so every seed asks for the same work."""
    r = random.Random("%(kind)s %(reqs)d %(len_lo)d %(len_hi)d" % {"len_lo": 0, "len_hi": 0, **c})
    lo, hi = (c["ctx_lo"], c["ctx_hi"]) if c["kind"] == "kv" else (c.get("len_lo", 0), c.get("len_hi", 0))
    one = c["kind"] in ("step", "replay") or (c["kind"] == "into" and c["sel"] in ("last", "slots"))
    n = [1 if one else r.randint(lo, hi) for _ in range(c["reqs"])]
    return [(t, not c.get("keep") or i % 2 == 0) for i, t in enumerate(n)]


def _rows(c, tokens):
    return -(-tokens // c.get("every", 1))


def _row_elems(c):
    return c["take"] * c["dim"] if c["kind"] == "kv" else c["width"]


def _geometry(c):
    """(rows of a record, its bytes, source bytes it reads, records of a pass)"""
    n = sum(_rows(c, t) for t, kept in _lengths(c) if kept)
    e = _row_elems(c)
    records = {"into": 1, "kv": 2 * c.get("layers", 0)}.get(c["kind"], c.get("points"))
    return n, B.record_bytes(c["reqs"], n, e, CODE[c["out"]], c["sums"]), n * e * SIZE[c["dtype"]], records


def work(case):
    n, record, read, records = _geometry(case)
    per = (2 if case["sums"] & 1 else 0) + (1 if case["sums"] & 2 else 0) + (1 if case["sums"] & 4 else 0)
    return {"bytes": float(records * (read + record + 20 * case["reqs"])), "flops": float(records * n * _row_elems(case) * per)}


def tolerance(case):
    # copies, gathers, downcasts and the layout are exact; norms and means are fp32 sums in some order
    return {"rel": 2e-6, "max": 2e-5} if case["sums"] & 3 else "exact"


# ------------------------------------------------------------------ inputs
def _values(gen, shape, dtype):
    """Activations: normal, with a few channels much larger than the rest, as residual streams have them."""
    x = torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16 if dtype != "fp32" else torch.float32)
    x[..., ::509] *= 30.0
    return x.to(TORCH[dtype])


def _inputs(c, seed):
    """Tensors, selection (one row per request: req_id, row_base, tok_start, tok_count, tok_step), keep vector,
    explicit rows, source row of every listed row."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    r = random.Random(seed)
    lens = _lengths(c)
    r.shuffle(lens)
    keep = [k for _, k in lens]
    sel = c.get("sel", "last")
    if c["kind"] == "kv":
        per = -(-c["ctx_hi"] // c["block"])
        shape = (c["seqs"] * per, c["block"], c["heads"], c["dim"])
        tensors = [_values(gen, shape, c["dtype"]) for _ in range(2 * c["layers"])]
        table = torch.randperm(c["seqs"] * per, generator=gen, device=DEV).to(torch.int32).view(c["seqs"], per)
        seqs = sorted(r.sample(range(c["seqs"]), c["reqs"]))
        reqs = [(9000 + q, q, 0, t, 1) for q, (t, _) in zip(seqs, lens)]
        heads = sorted(r.sample(range(c["heads"]), c["take"]))
        return {"tensors": tensors, "reqs": reqs, "table": table, "heads": heads, "keep": None, "index": None}
    if sel in ("last", "slots"):
        total = len(lens)
        at = list(range(total))
        if sel == "slots":
            r.shuffle(at)
        reqs = [(5000 + i, at[i], 0, 1, 1) for i in range(total)]
        rows = list(at)
    else:
        reqs, rows, total = [], [], 0
        for i, (t, _) in enumerate(lens):
            reqs.append((7000 + i, total, 0, _rows(c, t), c["every"]))
            rows += range(total, total + t, c["every"])
            total += t
    index = None
    if sel == "index":
        r.shuffle(rows)
        index = torch.tensor(rows, dtype=torch.int32, device=DEV)
    lead = c.get("lead", 0)     # a column slice of a wider matrix, which starts anywhere
    tensors = [_values(gen, (total, c["width"] + (lead + 8 if lead else 0)), c["dtype"])[:, lead:lead + c["width"]]
               for _ in range(c.get("points", 1))]
    return {"tensors": tensors, "reqs": reqs, "rows": rows, "index": index,
            "keep": torch.tensor(keep, dtype=torch.uint8, device=DEV) if c.get("keep") else None, "kept": keep}


class _Paged:
    def __init__(self, c, i):
        self.block_table, self.block_size, self.n_heads, self.head_dim = i["table"], c["block"], c["heads"], c["dim"]
        self.heads_sel = i["heads"]


def _round_up(n, to):
    return -(-n // to) * to


def _sections(c):
    """[(name, first byte, past the last byte, numpy type)] of a record, header included."""
    n, record, _, _ = _geometry(c)
    at = 64 + _round_up(16 * c["reqs"], 64)
    found = [("head", 0, at, np.uint32)]
    payload = _round_up(n * _row_elems(c) * SIZE[c["out"]], 64)
    if payload:
        found.append(("payload", at, at + payload, np.uint8))
    at += payload
    for name, bit in SUMS:
        if c["sums"] & bit:
            found.append((name, at, at + _round_up(4 * n, 64), np.float32))
            at += _round_up(4 * n, 64)
    assert at == record
    return found


# ------------------------------------------------------------------ the cases' state and one pass
def prepare(case, seed):
    c, i = case, _inputs(case, seed)
    n, record, _, records = _geometry(c)
    s = {"case": c, "inputs": i, "sections": _sections(c), "records": records, "bytes": record}
    if c["kind"] == "into":
        listed_rows = sum(q[3] for q in i["reqs"])
        s["out"] = torch.empty(B.record_bytes(c["reqs"], listed_rows, c["width"], CODE[c["out"]], c["sums"]),
                               dtype=torch.uint8, device=DEV)
        s["reqs"] = np.asarray(i["reqs"], dtype=np.uint32)
        kinds = {np.uint32: torch.int32, np.uint8: torch.uint8, np.float32: torch.float32}
        s["views"] = {k: s["out"][a:b].view(kinds[t]) for k, a, b, t in s["sections"]}
        return s
    # the device ring holds a few steps, the host ring two passes (or more, if they are tiny): one being
    # read, one arriving
    passes = max(2, -(-4096 // (record * records)))
    ring = B.Ring(max(1 << 20, _round_up(4 * record * records, 1 << 20)), passes * record * records,
                  max_reqs_per_observe=max(64, c["reqs"]))
    s["ring"], s["last"] = ring, -1
    how = {"out_dtype": CODE[c["out"]], "summary_mask": c["sums"]}
    if c["kind"] == "replay":
        ctx = H.StepContext()
        hooks = [H.HookPoint(ring, p, ctx, **how) for p in range(records)]
        graph = torch.cuda.CUDAGraph()
        gc.collect()        # what an earlier capture left behind frees its ring now, not inside this capture
        with ctx.capture(ring, i["reqs"], max_observes=records):
            with torch.cuda.graph(graph):
                for hook, x in zip(hooks, i["tensors"]):
                    hook(x)
        s.update(ctx=ctx, hooks=hooks, graph=graph)
    elif c["kind"] == "kv":
        s["calls"] = [B.PreparedBatch(ring, range(records), i["tensors"], i["reqs"], paged=_Paged(c, i), **how)]
    elif c["batch"]:
        s["calls"] = [B.PreparedBatch(ring, range(records), i["tensors"], i["reqs"], **how)]
    else:
        s["calls"] = [B.PreparedObserve(ring, p, x, i["reqs"], **how) for p, x in enumerate(i["tensors"])]
    return s


def run(state):
    c, stream = state["case"], torch.cuda.current_stream().cuda_stream
    if c["kind"] == "into":
        i = state["inputs"]
        B.observe_into(3, i["tensors"][0], state["reqs"], state["out"], seq=5, step_id=STEP_ID, out_dtype=CODE[c["out"]],
                       summary_mask=c["sums"], keep_mask=i["keep"], row_index=i["index"], stream=stream)
        return state["views"]
    ring, records = state["ring"], state["records"]
    if state["last"] >= 0:
        ring.release_host(state["last"])            # the previous pass has been read
    if c["kind"] == "replay":
        state["ctx"].begin_replay(STEP_ID, stream)
        state["graph"].replay()
        state["ctx"].end_replay(stream)
    else:
        for call in state["calls"]:
            code = call(STEP_ID, stream)
            if (code[0] if isinstance(code, tuple) else code) != B.OK:
                raise RuntimeError("observe: %r" % (code,))
    ring.drain(B.DRAIN_FLUSH)
    n, views = ring.poll_host_raw(records)
    # the host ring holds a whole number of passes, so a pass's records lie side by side in it
    if n != records or views[records - 1].p0 != views[0].p0 + (records - 1) * state["bytes"]:
        raise RuntimeError("%d records of %d arrived" % (n, records))
    state["last"] = views[records - 1].seq
    memory = (ctypes.c_uint8 * (records * state["bytes"])).from_address(views[0].p0)
    memory.owner = ring                             # the pinned memory lives as long as somebody reads it
    raw = np.frombuffer(memory, dtype=np.uint8).reshape(records, state["bytes"])
    got = {k: raw[:, a:b].view(t) for k, a, b, t in state["sections"]}
    head = got.pop("head")
    got["head"], got["seq"], got["rest"] = head[:, :2], head[:, 2] - head[0, 2], head[:, 4:]
    return got


# ------------------------------------------------------------------ the same in 64 bits
def exact(case, seed):
    c, i = case, _inputs(case, seed)
    n, _, read, records = _geometry(c)
    if c["kind"] == "kv":
        per = c["block"]
        tok = [(q[1], t) for q in i["reqs"] for t in range(q[3])]
        seq = torch.tensor([a for a, _ in tok], device=DEV)
        pos = torch.tensor([b for _, b in tok], device=DEV)
        block = i["table"][seq, pos // per].long()
        heads = torch.tensor(i["heads"], device=DEV)
        rows = [x[block, pos % per][:, heads].reshape(n, -1) for x in i["tensors"]]
    else:
        kept = [k for k, q in zip(i["kept"], i["reqs"]) for _ in range(q[3])]
        at = torch.tensor([r for r, k in zip(i["rows"], kept) if k], dtype=torch.long, device=DEV)
        rows = [x[at] for x in i["tensors"]]
    got = {name: [] for name, _ in SUMS}
    payload = []
    for x in rows:
        for a in range(0, n, 4096):
            y = x[a:a + 4096].double()
            got["l2"].append(y.square().sum(1).sqrt())
            got["mean"].append(y.mean(1))
            got["absmax"].append(y.abs().amax(1))
        if c["out"] != "none":
            y = x.float().clamp(-448.0, 448.0).to(torch.float8_e4m3fn) if c["out"] == "fp8" else x.to(TORCH[c["out"]])
            p = y.contiguous().view(torch.uint8).reshape(-1)
            payload.append(torch.nn.functional.pad(p, (0, _round_up(p.numel(), 64) - p.numel())).cpu())
    found = {"head": None}
    if c["out"] != "none":
        found["payload"] = payload[0] if c["kind"] == "into" else torch.stack(payload)
    for name, bit in SUMS:
        if c["sums"] & bit:
            v = torch.cat(got[name]).view(records, n)
            v = torch.nn.functional.pad(v, (0, _round_up(4 * n, 64) // 4 - n)).cpu()
            found[name] = v[0] if c["kind"] == "into" else v
    if c["kind"] != "into":
        found["seq"] = found["rest"] = None
    return found
