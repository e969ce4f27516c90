"""The attention calls that a user of this library makes, as cases to be timed and checked.

A case is one call of ``ops.prefill`` (question tokens over retrieved chunks), ``ops.decode`` (one new token per
request) or ``ops.decode_shared`` (the same, over a plan of the chunks that the batch's requests share).  The listed
cases are the shapes of this repository's benchmark and tests, together with the smaller, odd-sized and differently
laid out calls that surround them in a serving loop; ``draw`` spreads over the same ranges.

Fields of a case:
  kind      "prefill", "decode" or "shared"
  batch, hq, hkv, d, base   requests, query heads, KV heads, head dimension, RoPE base
  style     "half", "interleaved" (rotary pairing) or "alibi"
  keys      "nope" (keys stored unrotated) or "local" (keys stored at their local positions)
  scaled    True: a frequency table (long-context scaled RoPE) in place of the plain base
  prerot    True: queries arrive rotated
  prefix    keys of a prefix that every request shares (0: none)
  n_lo, n_hi, len_lo, len_hi   chunks per request and keys per chunk, uniform in the range
  pool      distinct stored chunks that the requests pick from without repetition; 0: private chunks
  zipf      popularity exponent of the pool's chunks (0: uniform)
  q_lo, q_hi   question tokens (prefill), or tokens generated so far (decode), uniform in the range
  block     tokens per block of a paged store (0: chunks are contiguous)
  order     "position" or "storage": order of a request's records in its table
  stream    True: the decode's non-temporal cache hint
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_04302_amd import ops

_CHUNK = np.dtype([("k_offset", "<i8"), ("v_offset", "<i8"), ("len", "<i4"), ("pos_offset", "<i4"),
                   ("k_stride", "<i4"), ("v_stride", "<i4")])

_DEFAULTS = dict(batch=1, hq=32, hkv=8, d=128, base=5.0e5, style="half", keys="nope", scaled=False, prerot=False,
                 prefix=0, n_lo=1, n_hi=1, len_lo=64, len_hi=64, pool=0, zipf=0.0, q_lo=1, q_hi=1, block=0,
                 order="position", stream=False)


def _case(kind, **kw):
    assert set(kw) <= set(_DEFAULTS) | {"name"}
    return dict(_DEFAULTS, kind=kind, **kw)


def listed():
    return [
        # The smallest call: a toy head layout, 272 keys, 16 question tokens.  Launch latency and host work.
        _case("prefill", name="tiny_prefill", hq=2, hkv=1, d=64, base=1.0e4, n_lo=4, n_hi=4, len_lo=64, len_hi=64,
              q_lo=16, q_hi=16),
        # One user's follow-up question over three retrieved passages of odd lengths: time to first token of a
        # single interactive request.
        _case("prefill", name="chat_prefill", prefix=128, n_lo=3, n_hi=3, len_lo=173, len_hi=811, q_lo=23, q_hi=23),
        # Short questions (a search box) of a batch: few query rows per request over several thousand keys.
        _case("prefill", name="short_question_prefill", batch=16, prefix=128, n_lo=5, n_hi=9, len_lo=200, len_hi=700,
              pool=96, q_lo=7, q_hi=48),
        # The benchmark's headline: eight requests, a shared prefix, ten 512-key chunks each from a pool of 64 and a
        # 64-token question.
        _case("prefill", name="rag_prefill", batch=8, prefix=128, n_lo=10, n_hi=10, len_lo=512, len_hi=512, pool=64,
              q_lo=64, q_hi=64),
        # The same work on a model with 64-wide heads and interleaved rotary pairs, odd chunk lengths.
        _case("prefill", name="rag_prefill_d64", batch=8, hkv=8, d=64, style="interleaved", prefix=100, n_lo=10,
              n_hi=10, len_lo=300, len_hi=700, pool=64, q_lo=101, q_hi=101),
        # One request over a long document in five parts, stored with local positions: the rotation-overhead shape.
        _case("prefill", name="long_document_prefill", keys="local", n_lo=5, n_hi=5, len_lo=4096, len_hi=4096,
              q_lo=64, q_hi=64),
        # Ragged batch: skewed chunk reuse, chunk lengths over a factor of 16, questions of 32 to 256 tokens, seven
        # query heads per KV head.
        _case("prefill", name="varlen_rag", batch=16, hq=28, hkv=4, base=1.0e6, n_lo=8, n_hi=24, len_lo=128,
              len_hi=2048, pool=200, zipf=2.1, q_lo=32, q_hi=256),
        # Many-shot in-context learning, the largest call: four requests, 128 exemplars each in their own order.
        _case("prefill", name="icl_prefill", batch=4, n_lo=128, n_hi=128, len_lo=256, len_hi=256, pool=128, q_lo=256,
              q_hi=256),
        # One user's next token over a paged store (64-token blocks): latency of a single decode stream.
        _case("decode", name="chat_decode", n_lo=5, n_hi=5, len_lo=301, len_hi=811, q_lo=37, q_hi=37, block=64),
        # A decode step of the in-context-learning batch.
        _case("decode", name="icl_decode", batch=4, n_lo=128, n_hi=128, len_lo=256, len_hi=256, pool=128, q_lo=300,
              q_hi=300),
        # The benchmark's decode batch: 64 requests, sixteen 1024-key chunks each from a pool of 256.
        _case("decode", name="rag_decode", batch=64, n_lo=16, n_hi=16, len_lo=1024, len_hi=1024, pool=256, q_lo=65,
              q_hi=65),
        # The same batch through the chunk-major plan that a server keeps for it.
        _case("shared", name="rag_decode_shared", batch=64, n_lo=16, n_hi=16, len_lo=1024, len_hi=1024, pool=256,
              q_lo=65, q_hi=65),
    ]


# ---------------------------------------------------------------------------------------------------------------
# Drawn cases.
# ---------------------------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "shared"])
    hq, hkv, d = rng.choice([(32, 8, 128), (32, 8, 128), (28, 4, 128), (32, 8, 64), (8, 8, 128), (40, 8, 128),
                             (12, 2, 64), (16, 1, 128)])
    style = rng.choice(["half", "half", "half", "interleaved", "alibi"])
    keys = "nope" if style == "alibi" else rng.choice(["nope", "nope", "local"])
    batch = _log(rng, 1, 64)
    n_hi = _log(rng, 1, 128)
    len_hi = _log(rng, 40, 4096)
    q_hi = _log(rng, 4, 400)
    c = _case(kind, batch=batch, hq=hq, hkv=hkv, d=d, base=rng.choice([1.0e4, 5.0e5, 1.0e6]), style=style, keys=keys,
              scaled=style != "alibi" and rng.random() < 0.25, prerot=style != "alibi" and rng.random() < 0.15,
              prefix=rng.choice([0, 0, 128, 77]), n_hi=n_hi, len_hi=len_hi, q_hi=q_hi,
              block=rng.choice([0, 0, 0, 64, 32]), order=rng.choice(["position", "position", "storage"]),
              stream=kind != "prefill" and rng.random() < 0.2)
    ragged = rng.random() < 0.6
    c["n_lo"] = max(1, n_hi // 3) if ragged else n_hi
    c["len_lo"] = max(1, len_hi // 8) if ragged else len_hi
    c["q_lo"] = max(1, q_hi // 6) if ragged else q_hi
    shared = kind == "shared" or rng.random() < 0.6

    # A drawn call costs no more than the largest listed one: shrink its longest ranges until it fits.
    def cost():
        keys_ = c["batch"] * (c["prefix"] + c["n_hi"] * c["len_hi"] + c["q_hi"])
        store = keys_ * c["hkv"] * c["d"] * 4
        flops = 4.0 * c["d"] * c["hq"] * keys_ * (c["q_hi"] if kind == "prefill" else 1)
        return max(store / 3.0e9, flops / 4.0e11)

    while cost() > 1:
        big = max(("batch", "n_hi"), key=lambda k: c[k]) if c["len_hi"] <= 256 else "len_hi"
        c[big] = max(1, int(c[big] * 0.71))
        c["n_lo"], c["len_lo"] = min(c["n_lo"], c["n_hi"]), min(c["len_lo"], c["len_hi"])
    c["pool"] = max(c["n_hi"], int(c["n_hi"] * rng.choice([1, 2, 6]))) if shared else 0
    c["zipf"] = rng.choice([0.0, 0.0, 1.5]) if shared else 0.0
    return c


# ---------------------------------------------------------------------------------------------------------------
# Inputs: a chunk store, one table of records per request, queries.  Values are N(0, 1) in bf16.
# ---------------------------------------------------------------------------------------------------------------
def _tables(case, seed):
    """(records, chunk_start, q_lens, q_pos0, elements of the store): host tables.  The lengths belong to the case;
    which chunks a request picks, their order and the places of a paged store's blocks come from the seed."""
    rng = np.random.default_rng([int(seed), 17])
    lens = np.random.default_rng([case[k] for k in ("batch", "n_lo", "n_hi", "len_lo", "len_hi", "q_lo", "q_hi")])
    per_key = case["hkv"] * case["d"]
    size = 0
    bt = case["block"]

    def store(n):
        """Place a chunk of n keys: its blocks as (first key, keys, K offset, V offset, stride)."""
        nonlocal size
        cuts = [(0, n, n)] if not bt else [(b, min(bt, n - b), bt) for b in range(0, n, bt)]
        got = []
        for first, keys, cap in cuts:
            got.append((first, keys, size, size + cap * per_key, cap))
            size += 2 * cap * per_key
        return n, got

    prefix = store(case["prefix"]) if case["prefix"] else None
    pool = [store(int(n)) for n in lens.integers(case["len_lo"], case["len_hi"] + 1, case["pool"])]
    p = None
    if pool and case["zipf"]:
        p = np.arange(1, len(pool) + 1, dtype=np.float64) ** -case["zipf"]
        p /= p.sum()
    uses, q_lens, q_pos0 = [], [], []
    for _ in range(case["batch"]):
        k = int(lens.integers(case["n_lo"], case["n_hi"] + 1))
        if pool:
            mine = [pool[i] for i in rng.permutation(rng.choice(len(pool), size=k, replace=False, p=p))]
        else:
            mine = [store(int(n)) for n in lens.integers(case["len_lo"], case["len_hi"] + 1, k)]
        uses.append(([prefix] if prefix else []) + mine)
        q_lens.append(int(lens.integers(case["q_lo"], case["q_hi"] + 1)))
    for u, n in zip(uses, q_lens):  # the question's (or the generated tokens') own keys
        q_pos0.append(sum(c[0] for c in u))
        u.append(store(n))
    if bt:  # a paged allocator's blocks lie in no particular order
        cap = 2 * bt * per_key
        where = rng.permutation(size // cap)
    recs, start = [], [0]
    for u in uses:
        pos = 0
        mine = []
        for n, blocks in u:
            for first, keys, ko, vo, cap_keys in blocks:
                if bt:
                    slot = int(where[ko // cap])
                    ko, vo = slot * cap, slot * cap + bt * per_key
                mine.append((ko, vo, keys, pos + first, cap_keys, cap_keys))
            pos += n
        if case["order"] == "storage":
            mine.sort(key=lambda r: r[0])
        recs += mine
        start.append(len(recs))
    return np.array(recs, dtype=_CHUNK), np.array(start, np.int32), q_lens, q_pos0, size


def _inputs(case, seed):
    recs, start, q_lens, q_pos0, size = _tables(case, seed)
    gen = torch.Generator("cuda").manual_seed(int(seed))
    pool = torch.empty(size, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    decode = case["kind"] != "prefill"
    if decode:  # one new token per request: the last of its tail, already in the store
        q_pos0 = [p + n - 1 for p, n in zip(q_pos0, q_lens)]
        q_lens = [1] * len(q_lens)
    q = torch.empty((sum(q_lens), case["hq"], case["d"]), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    table = None
    if case["scaled"]:  # frequencies below 1/1000 of a turn per position slowed by four, as long-context models do
        f = case["base"] ** (-2.0 * np.arange(case["d"] // 2) / case["d"])
        table = torch.from_numpy(np.where(f < 2 * math.pi / 1000, f / 4, f).astype(np.float32)).cuda()
    return dict(recs=recs, start=start, q_lens=q_lens, q_pos0=q_pos0, pool=pool, q=q, table=table)


def prepare(case, seed):
    x = _inputs(case, seed)
    i32 = lambda v: torch.tensor(np.asarray(v, np.int32), device="cuda")  # noqa: E731
    cfg = ops.Config(case["hq"], case["hkv"], case["d"], case["base"], inv_freq=x["table"],
                     key_positions=ops.KEYS_LOCAL if case["keys"] == "local" else ops.KEYS_NOPE,
                     rope_style={"half": ops.ROPE_HALF, "interleaved": ops.ROPE_INTERLEAVED,
                                 "alibi": ops.ALIBI}[case["style"]], q_prerotated=case["prerot"],
                     cache_hint=ops.CACHE_STREAM if case["stream"] else ops.CACHE_DEFAULT)
    keys = np.add.reduceat(x["recs"]["len"].astype(np.int64), x["start"][:-1])
    s = dict(kind=case["kind"], cfg=cfg, q=x["q"], q_pos0=i32(x["q_pos0"]), pool=x["pool"],
             max_kv=int(keys.max()), out=torch.empty_like(x["q"]),
             lse=torch.empty(x["q"].shape[:2], dtype=torch.float32, device="cuda"))
    if case["kind"] == "shared":
        s["plan"] = ops.upload_plan(ops.shared_decode_plan(cfg, x["recs"], x["start"]))
        nbytes = ops.decode_shared_workspace_size(cfg, case["batch"], s["plan"].max_slots)
    else:
        s["chunks"] = torch.from_numpy(x["recs"].view(np.uint8).copy()).cuda()
        s["chunk_start"] = i32(x["start"])
        if case["kind"] == "prefill":
            s["q_start"] = i32(np.concatenate([[0], np.cumsum(x["q_lens"])]))
            s["max_q"] = max(x["q_lens"])
            nbytes = ops.prefill_workspace_size(cfg, case["batch"], x["q"].shape[0], s["max_q"], s["max_kv"])
        else:
            nbytes = ops.decode_workspace_size(cfg, case["batch"], s["max_kv"])
    s["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
    return s


def run(s):
    if s["kind"] == "prefill":
        return ops.prefill(s["cfg"], s["q"], s["q_start"], s["q_pos0"], s["pool"], s["pool"], s["chunks"],
                           s["chunk_start"], s["max_q"], s["max_kv"], out=s["out"], lse=s["lse"],
                           workspace=s["workspace"])
    if s["kind"] == "decode":
        return ops.decode(s["cfg"], s["q"], s["q_pos0"], s["pool"], s["pool"], s["chunks"], s["chunk_start"],
                          s["max_kv"], out=s["out"], lse=s["lse"], workspace=s["workspace"])
    return ops.decode_shared(s["cfg"], s["q"], s["q_pos0"], s["pool"], s["pool"], s["plan"], out=s["out"],
                             lse=s["lse"], workspace=s["workspace"])


# ---------------------------------------------------------------------------------------------------------------
# What a call cannot do without, and what its outputs should be.
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    """Bytes: every stored key and value that some request reads, once, the tables, queries and outputs.  FLOPs: the
    two products over the visible (query, key) pairs."""
    recs, start, q_lens, q_pos0, _ = _tables(case, 0)
    decode = case["kind"] != "prefill"
    d, hq = case["d"], case["hq"]
    pairs = 0
    for r in range(case["batch"]):
        keys = int(recs["len"][start[r]:start[r + 1]].sum())
        n = q_lens[r]
        pairs += keys if decode else n * (keys - n) + n * (n + 1) // 2
    distinct = {(int(k), int(v)): int(n) for k, v, n in zip(recs["k_offset"], recs["v_offset"], recs["len"])}
    tokens = case["batch"] if decode else sum(q_lens)
    nbytes = sum(distinct.values()) * case["hkv"] * d * 4 + recs.nbytes + tokens * hq * (2 * 2 * d + 4)
    return {"bytes": float(nbytes), "flops": 4.0 * d * hq * pairs}


def tolerance(case):
    # bf16 inputs, fp32 sums.  Rotated keys, rotated queries, probabilities and outputs are each rounded to bf16;
    # against exact() the outputs of the listed and of sixteen drawn cases lie within 0.0038 (2-norm; largest single
    # difference 0.033) and their log-sum-exps within 1e-4.
    return {"rel": 1.5e-2, "max": 0.13}


def _rotate(x, pos, case, table):
    """x [..., n, d] rotated at positions pos [n], in 64 bits."""
    d = case["d"]
    f = table.double() if table is not None else \
        torch.pow(torch.tensor(case["base"], dtype=torch.float64, device=x.device),
                  -2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    a = pos.double()[:, None] * f
    c, s = torch.cos(a), torch.sin(a)
    if case["style"] == "interleaved":
        a1, a2 = x[..., 0::2], x[..., 1::2]
        return torch.stack([a1 * c - a2 * s, a1 * s + a2 * c], -1).flatten(-2)
    a1, a2 = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([a1 * c - a2 * s, a1 * s + a2 * c], -1)


def exact(case, seed):
    x = _inputs(case, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    G = hq // hkv
    dev = x["pool"].device
    out = torch.zeros(x["q"].shape, dtype=torch.float64, device=dev)
    lse = torch.zeros(x["q"].shape[:2], dtype=torch.float64, device=dev)
    t0 = 0
    for r in range(case["batch"]):
        n = x["q_lens"][r]
        qpos = x["q_pos0"][r] + torch.arange(n, device=dev)
        q = x["q"][t0:t0 + n].double().permute(1, 0, 2)  # [hq, n, d]
        if case["style"] != "alibi" and not case["prerot"]:
            q = _rotate(q, qpos, case, x["table"])
        ks, vs, kpos = [], [], []
        for rec in x["recs"][x["start"][r]:x["start"][r + 1]]:
            ko, vo, ln, pos, st, _ = (int(v) for v in rec)
            k = x["pool"][ko:ko + hkv * st * d].view(hkv, st, d)[:, :ln].double()
            p = pos + torch.arange(ln, device=dev)
            if case["style"] != "alibi":
                k = _rotate(k, p if case["keys"] == "nope" else torch.full_like(p, pos), case, x["table"])
            ks.append(k)
            vs.append(x["pool"][vo:vo + hkv * st * d].view(hkv, st, d)[:, :ln].double())
            kpos.append(p)
        k, v, kpos = torch.cat(ks, 1).contiguous(), torch.cat(vs, 1).contiguous(), torch.cat(kpos)
        kt = k.transpose(1, 2).contiguous()
        hidden = kpos[None, :] > qpos[:, None]
        for g in range(hkv):
            qg = q[g * G:(g + 1) * G]
            s = torch.matmul(qg.reshape(G * n, d).contiguous(), kt[g]).view(G, n, -1) / math.sqrt(d)
            if case["style"] == "alibi":
                h = torch.arange(g * G, (g + 1) * G, device=dev).double()
                s += torch.exp2(-8.0 * (h + 1) / hq)[:, None, None] * (kpos[None, :] - qpos[:, None]).double()
            s.masked_fill_(hidden, -math.inf)
            lse[t0:t0 + n, g * G:(g + 1) * G] = torch.logsumexp(s, -1).T
            o = torch.matmul(torch.softmax(s, -1).view(G * n, -1), v[g]).view(G, n, d)
            out[t0:t0 + n, g * G:(g + 1) * G] = o.permute(1, 0, 2)
        t0 += n
    return out, lse
