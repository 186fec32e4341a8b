"""The calls this library is used for, as cases that can be timed and compared.

A case is a dict of plain values.  Its "op" says which public entry points
one pass goes through:

  step     one serving step of the checkpoint loop: the newest tokens of every
           request are packed, and a step's rows are restored into another pool
           (issued as prepared calls, as a loop over fixed buffers does).
           "via": "ranges" (one launch per copy) or "plan" (plan, then copies).
  full     plan and pack of every request's whole context
  restore  plan and unpack of whole contexts into a partly occupied pool
  recover  a restore in validate mode: plan, validate_targets, status (the
           host decides on it), unpack
  to_host  plan and pack_to_host of a step, through a staging ring
  draft    draft-state alignment of a batch

The other fields: the cache ("layers", "heads", "dim", "block", "order",
"elem" bytes per element), "reqs" requests of "lo" to "hi" planned tokens,
"ctx" the median context in front of them (0: from position 0), "rows"
("packed", or "regions" with one reserved checkpoint region per request), and
"arena", how many steps' rows the checkpoint buffer holds (the copies are
given the whole buffer, as a serving loop that allocates it once does).

Token counts and contexts are the quantiles of their distribution, dealt to
the requests in an order the seed draws, so the work of a case does not
depend on the seed; block tables are random permutations of the pool and the
contents are N(0,1) values (random bytes for 1-byte caches).  Every output is
raw copied bits or whole numbers, so results are compared exactly.
"""
from __future__ import annotations

import math
import statistics

import numpy as np
import torch

import paper_2606_17787_amd.kvckpt as kv
from paper_2606_17787_amd.workloads import CacheShape

_LLAMA_8B = dict(layers=32, heads=8, dim=128, block=16, order="NHD", elem=2)
_LLAMA_70B_TP8 = dict(layers=80, heads=1, dim=128, block=16, order="NHD",
                      elem=2)
_QWEN_HND = dict(layers=28, heads=4, dim=128, block=32, order="HND", elem=2)
_TINY = dict(layers=2, heads=2, dim=64, block=16, order="NHD", elem=2)


def listed():
    return [
        # The smallest call: every request of a tiny cache packed whole and
        # restored under a new table; launches and host calls are all it is.
        dict(_TINY, name="tiny-roundtrip", op="step", via="plan",
             rows="packed", reqs=8, lo=100, hi=300, ctx=0, arena=1),
        # A lightly loaded worker: 8 requests append a few tokens each to
        # their reserved regions of a checkpoint arena (speculative decoding
        # commits several tokens a step).
        dict(_LLAMA_8B, name="small-step-regions", op="step", via="ranges",
             rows="regions", reqs=8, lo=1, hi=16, ctx=700, arena=16),
        # Plain decoding: one new token per request and step, packed rows.
        dict(_LLAMA_8B, name="decode-1-token", op="step", via="ranges",
             rows="packed", reqs=48, lo=1, hi=1, ctx=700, arena=20),
        # The headline step: 256 requests, 1-16 new tokens each.
        dict(_LLAMA_8B, name="decode-256", op="step", via="ranges",
             rows="packed", reqs=256, lo=1, hi=16, ctx=512, arena=4),
        # The same step with a region per request, as plan + copies.
        dict(_LLAMA_8B, name="decode-256-regions", op="step", via="plan",
             rows="regions", reqs=256, lo=1, hi=16, ctx=512, arena=2),
        # A head-major cache with short runs: the copy transposes.
        dict(_QWEN_HND, name="qwen-step", op="step", via="ranges",
             rows="packed", reqs=200, lo=1, hi=64, ctx=400, arena=2),
        # An 8-bit cache (the serving option that halves the KV), whole
        # contexts of odd lengths, packed and restored.
        dict(_QWEN_HND, name="fp8-hnd-roundtrip", op="step", via="plan",
             rows="packed", reqs=13, lo=311, hi=2777, ctx=0, arena=1) |
        dict(elem=1),
        # A first checkpoint: one tensor-parallel rank's whole contexts.
        dict(_LLAMA_70B_TP8, name="tp8-full-pack", op="full", via="plan",
             rows="packed", reqs=24, lo=500, hi=8000, ctx=0, arena=1),
        # A failure's burst of restores into fragmented free blocks.
        dict(_LLAMA_8B, name="restore-burst", op="restore", via="plan",
             rows="packed", reqs=5, lo=1024, hi=6000, ctx=0, arena=1),
        # One interrupted request of a tensor-parallel rank, validated first.
        dict(_LLAMA_70B_TP8, name="recover-one", op="recover", via="plan",
             rows="packed", reqs=1, lo=2003, hi=2003, ctx=0, arena=1),
        # The background checkpoint to pinned host memory.
        dict(_LLAMA_8B, name="step-to-host", op="to_host", via="plan",
             rows="packed", reqs=32, lo=1, hi=16, ctx=700, arena=1),
        # A recovering worker aligns its draft KV after a progress update.
        dict(name="draft-align", op="draft", reqs=1024, lo=1024, hi=4096,
             depth=4, block=16),
    ]


# ------------------------------------------------------------------ drawing

_MOST_BYTES = 4.0e9   # checkpoint bytes of a drawn case
_MOST_POOL = 20.0e9   # source pool bytes of a drawn case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "full", "restore",
                     "recover", "to_host", "draft"])
    if op == "draft":
        lo = _log(rng, 64, 2048)
        return dict(op=op, reqs=_log(rng, 4, 1024), lo=lo,
                    hi=lo + _log(rng, 16, 2048), depth=rng.randint(1, 8),
                    block=rng.choice([16, 32]))
    c = dict(rng.choice([_LLAMA_8B, _LLAMA_8B, _LLAMA_70B_TP8, _QWEN_HND,
                         _TINY]))
    c["order"] = rng.choice([c["order"], c["order"], "NHD", "HND"])
    c["elem"] = rng.choice([2, 2, 2, 1, 4])
    c["block"] = rng.choice([c["block"], c["block"], 16, 32, 64])
    c["op"], c["via"], c["rows"], c["arena"], c["ctx"] = (op, "plan", "packed",
                                                          1, 0)
    rb = _row_bytes(c)
    if op in ("step", "to_host"):
        most = min(256, max(2, int(_MOST_POOL / rb / 700)))
        c["reqs"] = _log(rng, 1, most)
        c["lo"] = 1
        c["hi"] = rng.choice([1, rng.randint(2, 16), rng.randint(17, 64)])
        c["ctx"] = _log(rng, 100, 700)
        if op == "to_host":
            c["hi"] = min(c["hi"], max(1, int(2e8 / rb / c["reqs"])))
        else:
            c["via"] = rng.choice(["ranges", "ranges", "plan"])
            c["rows"] = rng.choice(["packed", "regions"])
            c["arena"] = rng.choice([1, 2, 4, 16])
            while (c["arena"] > 1 and
                   c["arena"] * c["reqs"] * c["hi"] * rb > _MOST_BYTES):
                c["arena"] //= 2
            while c["reqs"] > 1 and c["reqs"] * c["hi"] * rb > _MOST_BYTES:
                c["reqs"] //= 2
    else:
        c["reqs"] = 1 if op == "recover" else _log(rng, 1, 40)
        top = max(4, int(0.4 * _MOST_BYTES / rb / c["reqs"]))
        c["hi"] = _log(rng, min(64, top // 2), min(top, 12000))
        c["lo"] = max(1, int(c["hi"] * rng.uniform(0.1, 1.0)))
    return c


# ---------------------------------------------------------------- the inputs

def _shape(c):
    return CacheShape(c["layers"], c["heads"], c["dim"], c["block"],
                      c["order"], c["elem"])


def _row_bytes(c):
    return c["layers"] * 2 * c["heads"] * c["dim"] * c["elem"]


def _tokens(c):
    """Planned tokens per request: evenly spread over [lo, hi]."""
    R, lo, hi = c["reqs"], c["lo"], c["hi"]
    return [lo + int((hi - lo + 1) * (i + 0.5) / R) for i in range(R)]


def _contexts(c):
    """Quantiles of a lognormal context length (sigma 0.75) around "ctx"."""
    R, mid = c["reqs"], c["ctx"]
    if not mid:
        return [0] * R
    z = statistics.NormalDist()
    return [max(1, min(8 * mid, int(round(mid * math.exp(
        0.75 * z.inv_cdf((i + 0.5) / R)))))) for i in range(R)]


_DTYPE = {1: torch.uint8, 2: torch.int16, 4: torch.int32}


def _noise(n, elem, gen):
    """n elements of cache contents: N(0,1) as bf16 or fp32, or bytes."""
    if elem == 1:
        words = torch.empty(-(-n // 8), dtype=torch.int64, device="cuda")
        return words.random_(generator=gen).view(torch.uint8)[:n]
    dt = torch.bfloat16 if elem == 2 else torch.float32
    x = torch.empty(n, dtype=dt, device="cuda")
    return x.normal_(generator=gen).view(_DTYPE[elem])


def _tables(rng, num_blocks, first, end, free=None):
    """Pages [first, end) of every request take blocks of a permutation."""
    perm = (rng.permutation(num_blocks) if free is None else free)
    bt = np.full((len(first), int(end.max())), -1, np.int32)
    pos = 0
    for r, (a, b) in enumerate(zip(first, end)):
        bt[r, a:b] = perm[pos:pos + b - a]
        pos += b - a
    return bt


def _cuda(a, dtype=np.int32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


def _prepare_draft(c, seed):
    R, depth, bs = c["reqs"], c["depth"], c["block"]
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    hist = rng.permutation(np.array(_tokens(c), np.int64))
    cols = int(max(_tokens(c))) + depth + 1
    draft = torch.empty(R, cols, dtype=torch.int32, device="cuda")
    draft.random_(0, 128256, generator=gen)
    committed = draft.clone()
    accepted = rng.integers(0, depth + 1, R)
    at = torch.from_numpy(hist + accepted).cuda()
    committed[torch.arange(R, device="cuda"), at] += 1  # the correction
    pages = -(-cols // bs)
    # KV lengths and tables as the draft step left them, in one buffer each.
    before = torch.cat([
        _cuda(hist + depth), _cuda(rng.permutation(R * pages))])
    now = before.clone()
    return dict(
        c=c, draft=draft, committed=committed, dl=_cuda(hist + depth),
        cl=_cuda(hist + accepted + 1), before=before, now=now,
        kv_len=now[:R], tables=now[R:].view(R, pages),
        replay=torch.zeros(R, dtype=torch.int32, device="cuda"),
        freed=torch.zeros(R * (depth // bs + 2), dtype=torch.int32,
                          device="cuda"),
        count=torch.zeros(1, dtype=torch.int64, device="cuda"),
        ws=kv.new_workspace(R, "cuda"))


def prepare(case, seed):
    c = dict(case)
    c.pop("name", None)
    if c["op"] == "draft":
        return _prepare_draft(c, seed)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    sh, bs, R = _shape(c), c["block"], c["reqs"]
    start = rng.permutation(np.array(_contexts(c), np.int64))
    end = start + rng.permutation(np.array(_tokens(c), np.int64))
    total = int((end - start).sum())
    pages, touched = -(-end // bs), start // bs
    zero = np.zeros(R, np.int64)
    st = dict(c=c, sh=sh, total=total, start=_cuda(start), end=_cuda(end))

    base, rrb = 0, None
    if c["rows"] == "packed":
        rows = c["arena"] * total
        base = (c["arena"] // 2) * total
    else:
        room = c["arena"] * c["hi"]
        rows = R * room
        rrb = np.arange(R) * room + (c["arena"] // 2) * c["hi"] - start
        rrb = _cuda(rrb, np.int64)
    packs = c["op"] in ("step", "full", "to_host")
    if packs:
        st["src_nb"] = int(pages.sum())
        st["src"] = _noise(sh.pool_elems(st["src_nb"]), c["elem"], gen)
        st["bt"] = _cuda(_tables(rng, st["src_nb"], zero, pages))
    if c["op"] == "step":
        # room for a step of the longest deltas, however they meet the pages
        st["dst_nb"] = R * ((c["hi"] - 1) // bs + 2)
        st["bt2"] = _cuda(_tables(rng, st["dst_nb"], touched, pages))
    elif c["op"] in ("restore", "recover"):
        # 60% of the pool belongs to other requests
        st["dst_nb"] = -(-int(pages.sum()) * 5 // 2)
        free = rng.permutation(st["dst_nb"])[:int(pages.sum())]
        st["bt2"] = _cuda(_tables(rng, st["dst_nb"], zero, pages, free))
    if "dst_nb" in st:
        st["dst"] = torch.zeros(sh.pool_elems(st["dst_nb"]),
                                dtype=_DTYPE[c["elem"]], device="cuda")
    row = sh.token_row_elems
    if c["op"] in ("restore", "recover"):
        st["ckpt"] = _noise(rows * row, c["elem"], gen)
    elif c["op"] != "to_host":
        st["ckpt"] = torch.zeros(rows * row, dtype=_DTYPE[c["elem"]],
                                 device="cuda")

    if c["op"] == "step" and c["via"] == "ranges":
        st["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        st["calls"] = [
            kv.prepare_pack_ranges(sh, st["src_nb"], st["src"], st["bt"],
                                   st["start"], st["end"], st["ckpt"],
                                   st["status"], base, rrb),
            kv.prepare_unpack_ranges(sh, st["dst_nb"], st["dst"], st["bt2"],
                                     st["start"], st["end"], st["ckpt"],
                                     st["status"], base, rrb)]
        return st
    st["ws"] = kv.new_workspace(R, "cuda")
    if c["op"] == "step":
        st["calls"] = [
            kv.prepare_plan(st["start"], st["end"], st["ws"], base, rrb),
            kv.prepare_pack(sh, st["src_nb"], st["src"], st["bt"], st["ws"],
                            st["ckpt"]),
            kv.prepare_unpack(sh, st["dst_nb"], st["dst"], st["bt2"],
                              st["ws"], st["ckpt"])]
    elif c["op"] == "recover":
        st["marks"] = kv.new_marks(st["dst_nb"], "cuda")
    elif c["op"] == "to_host":
        st["slots"] = 2
        slot_rows = max(1, min(128, -(-total // 2)))
        st["staging"] = torch.empty(st["slots"] * slot_rows *
                                    sh.token_row_bytes, dtype=torch.uint8,
                                    device="cuda")
        st["host"] = torch.zeros(total * sh.token_row_bytes,
                                 dtype=torch.uint8, pin_memory=True)
        st["pack_s"], st["copy_s"] = torch.cuda.Stream(), torch.cuda.Stream()
    return st


# ----------------------------------------------------------------- one pass

def run(st):
    op = st["c"]["op"]
    if op == "draft":
        # the draft step before it grew every KV by the proposed tokens
        st["now"].copy_(st["before"])
        kv.lumen_kv_draft_align(st["draft"], st["dl"], st["committed"],
                                st["cl"], st["kv_len"], st["tables"],
                                st["c"]["block"], st["replay"], st["freed"],
                                st["count"], st["ws"])
        return [st["now"], st["replay"], st["freed"], st["count"]]
    if op == "step":
        for call in st["calls"]:
            call()
        return [st["ckpt"], st["dst"]]
    if op == "to_host":
        kv.lumen_kv_ckpt_plan(st["start"], st["end"], st["ws"],
                              stream=st["pack_s"])
        kv.lumen_kv_ckpt_pack_to_host(
            st["sh"], st["src_nb"], st["src"], st["bt"], st["ws"],
            st["total"], st["staging"], st["slots"], st["host"],
            pack_stream=st["pack_s"], copy_stream=st["copy_s"])
        return st["host"]
    kv.lumen_kv_ckpt_plan(st["start"], st["end"], st["ws"])
    if op == "full":
        kv.lumen_kv_ckpt_pack(st["sh"], st["src_nb"], st["src"], st["bt"],
                              st["ws"], st["ckpt"])
        return st["ckpt"]
    code = 0
    if op == "recover":
        kv.lumen_kv_ckpt_validate_targets(st["sh"], st["dst_nb"], st["bt2"],
                                          st["ws"], st["marks"])
        code = kv.lumen_kv_ckpt_status(st["ws"])
    if code == kv.LUMEN_OK:
        kv.lumen_kv_ckpt_unpack(st["sh"], st["dst_nb"], st["dst"], st["bt2"],
                                st["ws"], st["ckpt"])
    return [st["dst"], code]


# ------------------------------------------------------ what a pass has to do

def work(case):
    """Bytes read and written once: the planned rows on either side of each
    copy, the ranges and the touched block-table entries; for the draft
    alignment the tokens up to each request's mismatch, the lengths, and the
    KV state its pass starts from."""
    c = case
    R, n = c["reqs"], _tokens(c)
    if c["op"] == "draft":
        pages = -(-(max(n) + c["depth"] + 1) // c["block"])
        tokens = sum(n) + R * (c["depth"] / 2 + 1)
        return {"bytes": 8.0 * tokens + 2 * 4.0 * R * (pages + 1) + 20.0 * R,
                "flops": 0.0}
    copies = 2 if c["op"] == "step" else 1
    table = 4.0 * (sum(n) / c["block"] + R)
    return {"bytes": copies * (2.0 * sum(n) * _row_bytes(c) + table + 8.0 * R),
            "flops": 0.0}


def tolerance(case):
    """Copied bits and whole numbers."""
    return "exact"


def exact(case, seed):
    """No output is a computed number with a rounding."""
    return None
