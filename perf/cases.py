"""Workloads of the mixed action+decode attention path, through the C ABI's Python binding.

One case is one pass of what a serving program does over and over: a whole attention step (batch
descriptor, then append and attention of every layer), the layers of a step whose descriptor is
already built, the start of a frame (the observation's prefill cache is stored, the tasks fan out
and run their first step), or a request's history loaded and read back.

Geometry is the library's: 8 query heads over one KV head, head_dim 256, pages of 16 tokens, bf16.
Keys, values and queries are N(0, 1) with softmax scale 1/16; pool blocks are handed out in a
shuffled order, as in a pool that has been in use for a while.
"""
import math
import random

import torch

from paper_2603_14371_amd import binding as B

HEADS, DIM, PAGE = 8, 256, 16
SCALE = 1.0 / 16.0
ROW = DIM * 2                    # bytes of one key or value row


def _case(name, kind, **kw):
    """kind: "step" = one whole step, batch descriptor included; "layers" = the layers of a step
    whose descriptor is in hand, one call per layer; "start" = prefill cache stored, fan-out, first
    step, release; "reload" = histories loaded append-only and read back.
    prefixes x prefix_len observations; chunks action chunks of chunk_len queries (chunk i on
    observation i, counted round); decoders requests with own histories of hist_lo..hist_hi tokens
    and n_new new tokens each (request i on observation i // ceil(decoders / prefixes)).
    form: "fold" = append inside the attention's launches, "graph" = the same replayed from a
    recording, "separate" = append, then attention."""
    c = dict(kind=kind, layers=18, prefixes=1, prefix_len=832, chunks=0, chunk_len=50, decoders=0,
             hist_lo=1, hist_hi=1, n_new=1, form="fold", lse=False, lengths=1)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one layer, a 64-token observation, a chunk of 10 and a request
        _case("tiny_step", "step", layers=1, prefix_len=64, chunks=1, chunk_len=10, decoders=1,
              hist_lo=4, hist_hi=4, form="separate", lse=True),
        # a frame begins: prefill cache of one observation stored in all layers, action and
        # language streams created, their first step, everything released again
        _case("frame_start", "start", chunks=1, decoders=1, hist_lo=0, hist_hi=0),
        # one denoise step of the frame's chunk together with one decode token
        _case("frame_mixed_step", "step", chunks=1, decoders=1, hist_lo=9, hist_hi=9),
        # the decode loop after the denoise steps
        _case("frame_decode_step", "step", decoders=1, hist_lo=40, hist_hi=40),
        # eight requests of earlier frames (each on its own observation) and the new frame's chunk
        _case("cross_frame_step", "step", prefixes=8, chunks=1, decoders=8, hist_lo=16,
              hist_hi=512, lengths=2),
        # narration, memory and planning decode together on one observation, replayed
        _case("cross_task_decode", "step", decoders=3, hist_lo=60, hist_hi=380, form="graph",
              lengths=3),
        # chunks of eight robots' observations, no language: the dense side, layer by layer
        _case("chunks_832_layers", "layers", layers=6, prefixes=8, chunks=8),
        _case("chunks_2048_layers", "layers", layers=6, prefixes=8, prefix_len=2048, chunks=8),
        # several tokens per request at once, causal (parallel decoding, draft verification),
        # ragged everywhere
        _case("verify_layers", "layers", layers=6, prefixes=3, prefix_len=771, decoders=6,
              hist_lo=30, hist_hi=900, n_new=13, form="separate", lse=True, lengths=4),
        # 64 requests in groups of eight on long observations, two chunks
        _case("stress_step", "step", prefixes=8, prefix_len=2048, chunks=2, decoders=64, hist_lo=1,
              hist_hi=2048, lengths=5),
        # the same geometry four times as wide, fewer layers
        _case("wide_step", "step", layers=5, prefixes=32, prefix_len=2048, chunks=2, decoders=256,
              hist_lo=1, hist_hi=2048, lengths=6),
        # histories of four requests brought into the pool and read back (a request that moves)
        _case("history_reload", "reload", layers=6, prefixes=0, decoders=4, hist_lo=100,
              hist_hi=700, lengths=7),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    """Steps of every mixture: observations of 16..2048 tokens, up to 16 of them, up to 64
    requests with histories up to 2048 tokens, up to eight chunks of 3..64 queries, one or
    several new tokens per request, either call form."""
    kind = rng.choice(["step", "step", "step", "layers", "layers", "start", "reload"])
    hi = _log_int(rng, 8, 2048)
    c = dict(layers=rng.randint(1, 18), prefixes=_log_int(rng, 1, 16),
             prefix_len=_log_int(rng, 16, 2048), chunk_len=rng.randint(3, 64), hist_hi=hi,
             hist_lo=rng.randint(1, hi), lse=rng.random() < 0.3, lengths=rng.randint(100, 1 << 20),
             form=rng.choice(["fold", "fold", "fold", "graph", "separate"]))
    if kind == "reload":
        c.update(prefixes=0, decoders=_log_int(rng, 1, 8), layers=rng.randint(1, 6), form="fold")
        return _case(None, kind, **c)
    if kind == "start":
        c.update(prefixes=1, chunks=1, decoders=rng.randint(0, 3), hist_lo=0, hist_hi=0)
        return _case(None, kind, **c)
    mix = rng.choice(["mixed", "mixed", "decode", "chunks"])
    if mix != "chunks":
        c["decoders"] = _log_int(rng, 1, 64)
        if rng.random() < 0.25:
            c["n_new"] = rng.randint(2, 16)
            c["decoders"] = min(c["decoders"], 12)
    if mix != "decode":
        c["chunks"] = rng.randint(1, min(8, c["prefixes"]))
    if kind == "layers" and c["form"] == "graph":
        c["form"] = "fold"
    c = _case(None, kind, **c)
    tokens = c["prefixes"] * c["prefix_len"] + sum(_histories(c))
    c["layers"] = max(1, min(c["layers"], 1400000 // tokens))
    return c


def _histories(case):
    rng = random.Random(case["lengths"])
    return [rng.randint(case["hist_lo"], case["hist_hi"]) for _ in range(case["decoders"])]


def _prefix_of(case, i):
    """Observation of request i (-1: none)."""
    if case["prefixes"] == 0:
        return -1
    return i // -(-case["decoders"] // case["prefixes"])


def _items(case):
    """(observation, own history, new tokens, bidirectional) of every item, in batch order."""
    items = [(i % max(1, case["prefixes"]), 0, case["chunk_len"], True)
             for i in range(case["chunks"])]
    items += [(_prefix_of(case, i), h, case["n_new"], False)
              for i, h in enumerate(_histories(case))]
    return items


def _normal(seed, tag, layer, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + tag) * 64 + layer)
    return torch.randn(shape, device="cuda", generator=g).to(torch.bfloat16)


def _prefix_rows(case, seed, i, layer):
    """K and V of observation i in one layer: [2, prefix_len, 256]."""
    return _normal(seed, 10 + i, layer, 2, case["prefix_len"], DIM)


def _history_rows(case, seed, layer):
    """K and V of all requests' histories in one layer, one after the other."""
    return _normal(seed, 1, layer, 2, sum(_histories(case)), DIM)


def _step_rows(case, seed, layer):
    """New K and V rows and queries of the step in one layer."""
    n = sum(it[2] for it in _items(case))
    return _normal(seed, 2, layer, 2, n, DIM), _normal(seed, 3, layer, n, HEADS, DIM)


class _State:
    """A pool with its streams, and the step's resident inputs and outputs."""

    def __init__(self, case, seed):
        self.case = case
        self.pool = self.batch = None
        L = case["layers"]
        self.items = _items(case)
        hist = _histories(case)
        pages = lambda n: -(-n // PAGE)  # noqa: E731
        blocks = case["prefixes"] * pages(case["prefix_len"])
        blocks += sum(pages(h + n) for _, h, n, _ in self.items) + 64
        order = list(range(blocks))
        random.Random(seed).shuffle(order)
        n_q = sum(n for _, _, n, _ in self.items)
        cfg = B.make_config(L, blocks, free_order=order, max_live_batches=2,
                            max_q_tokens=max(16, n_q), max_append_tokens=max(16, n_q, sum(hist)))
        self.kv = torch.empty(B.oxy_kv_bytes(cfg), dtype=torch.uint8, device="cuda")
        self.ws = torch.empty(B.oxy_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
        cfg.kv_base, cfg.kv_bytes = self.kv.data_ptr(), self.kv.numel()
        cfg.workspace, cfg.workspace_bytes = self.ws.data_ptr(), self.ws.numel()
        self.pool = B.oxy_pool_create(cfg)
        self.stream = torch.cuda.current_stream().cuda_stream
        if case["kind"] == "reload":
            rows = [_history_rows(case, seed, l) for l in range(L)]
            self.kv_new = torch.stack(rows)                         # [L, 2, n, 256]
            self.kv_back = torch.empty_like(self.kv_new)
            self.hist = hist
            return
        if case["kind"] == "start":
            rows = [_prefix_rows(case, seed, 0, l) for l in range(L)]
            self.prefill = torch.stack(rows).transpose(0, 1).contiguous()   # [2, L, P, 256]
        else:
            self._load(seed, hist)
        kv, q = zip(*[_step_rows(case, seed, l) for l in range(L)])
        self.kv_new = torch.stack(kv).transpose(0, 1).contiguous()  # [2, L, n, 256]
        self.q = torch.stack(q)                                     # [L, n, 8, 256]
        self.out = torch.empty_like(self.q)
        self.lse = torch.empty((L, n_q, HEADS), device="cuda") if case["lse"] else None
        if case["kind"] == "layers":
            self.batch = B.oxy_batch_build(self.pool, self.batch_items, 0, self.stream)

    def _load(self, seed, hist):
        case, pool, s = self.case, self.pool, self.stream
        L, P = case["layers"], case["prefix_len"]
        pids = [B.oxy_prefix_create(pool) for _ in range(case["prefixes"])]
        for i, pid in enumerate(pids):
            for l in range(L):
                kv = _prefix_rows(case, seed, i, l)
                B.oxy_prefix_append(pool, pid, l, kv[0].data_ptr(), kv[1].data_ptr(), P, 0, s)
        sids = [B.oxy_stream_create(pool, pids[p], B.KIND_ACTION if both else B.KIND_DECODE)
                for p, _, _, both in self.items]
        self.batch_items = [(sid, it[2]) for sid, it in zip(sids, self.items)]
        self.rewinds = [(sid, it[1]) for sid, it in zip(sids, self.items) if not it[3]]
        if hist:
            b = B.oxy_batch_build(pool, self.rewinds, B.BATCH_APPEND_ONLY, s)
            for l in range(L):
                kv = _history_rows(case, seed, l)
                B.oxy_stream_append(pool, b, l, kv[0].data_ptr(), kv[1].data_ptr(), s)
            B.oxy_batch_destroy(b)

    def close(self):
        if self.pool is not None:
            torch.cuda.synchronize()
            if self.batch is not None:
                B.oxy_batch_destroy(self.batch)
            B.oxy_pool_destroy(self.pool)
            self.pool = None

    def __del__(self):
        self.close()

    def results(self):
        return {"out": self.out} if self.lse is None else {"out": self.out, "lse": self.lse}


def prepare(case, seed):
    return _State(case, seed)


def _run_layers(s, batch):
    """One call per layer (two with a separate append), as a model's layers make them."""
    k, v, q, o, lse = s.kv_new[0], s.kv_new[1], s.q, s.out, s.lse
    for l in range(s.case["layers"]):
        kp, vp = k[l].data_ptr(), v[l].data_ptr()
        lp = 0 if lse is None else lse[l].data_ptr()
        if s.case["form"] == "separate":
            B.oxy_stream_append(s.pool, batch, l, kp, vp, s.stream)
            B.oxy_mixed_attention(s.pool, batch, l, q[l].data_ptr(), o[l].data_ptr(), lp, SCALE,
                                  s.stream)
        else:
            B.oxy_append_attention(s.pool, batch, l, kp, vp, q[l].data_ptr(), o[l].data_ptr(), lp,
                                   SCALE, s.stream)


def _run_step(s, items):
    """Batch descriptor, then all layers in one call."""
    flags = {"fold": B.STEP_FOLD_APPEND, "graph": B.STEP_FOLD_APPEND | B.STEP_GRAPH,
             "separate": 0}[s.case["form"]]
    n, L = s.q.shape[1], s.case["layers"]
    batch = B.oxy_batch_build(s.pool, items, 0, s.stream)
    B.oxy_step_layers(s.pool, batch, 0, L, s.kv_new[0].data_ptr(), s.kv_new[1].data_ptr(), n * ROW,
                      s.q.data_ptr(), s.out.data_ptr(), n * HEADS * ROW,
                      0 if s.lse is None else s.lse.data_ptr(), n * HEADS * 4, SCALE, flags, None,
                      s.stream)
    B.oxy_batch_destroy(batch)


def run(s):
    case = s.case
    if case["kind"] == "layers":
        _run_layers(s, s.batch)
        return s.results()
    if case["kind"] == "step":
        for sid, length in s.rewinds:      # the same step again: drop the tokens it appended
            B.oxy_stream_rewind(s.pool, sid, length)
        _run_step(s, s.batch_items)
        return s.results()
    if case["kind"] == "start":
        P, L = case["prefix_len"], case["layers"]
        pid = B.oxy_prefix_create(s.pool)
        B.oxy_prefix_append_layers(s.pool, pid, 0, L, s.prefill[0].data_ptr(),
                                   s.prefill[1].data_ptr(), P * ROW, P, 0, s.stream)
        sids = [B.oxy_stream_create(s.pool, pid, B.KIND_ACTION if it[3] else B.KIND_DECODE)
                for it in s.items]
        _run_step(s, [(sid, it[2]) for sid, it in zip(sids, s.items)])
        for sid in sids:
            B.oxy_stream_release(s.pool, sid)
        B.oxy_prefix_release(s.pool, pid)
        return s.results()
    sids = [B.oxy_stream_create(s.pool, -1, B.KIND_DECODE) for _ in s.hist]
    batch = B.oxy_batch_build(s.pool, list(zip(sids, s.hist)), B.BATCH_APPEND_ONLY, s.stream)
    slots = B.oxy_batch_slots(batch)
    for l in range(case["layers"]):
        B.oxy_stream_append(s.pool, batch, l, s.kv_new[l, 0].data_ptr(), s.kv_new[l, 1].data_ptr(),
                            s.stream)
        B.oxy_gather_kv(s.pool, l, slots, s.kv_back[l, 0].data_ptr(), s.kv_back[l, 1].data_ptr(),
                        s.stream)
    B.oxy_batch_destroy(batch)
    for sid in sids:
        B.oxy_stream_release(s.pool, sid)
    return {"kv": s.kv_back}


def _visible(case):
    """Sum over queries of the tokens each one sees."""
    total = 0
    for p, h, n, both in _items(case):
        pre = case["prefix_len"] if p >= 0 else 0
        total += n * (pre + n) if both else n * (pre + h) + n * (n + 1) // 2
    return total


def work(case):
    """Live keys and values read once, new rows read and stored once, queries read, outputs
    written; 4 * 256 flops per (query row, key)."""
    L = case["layers"]
    if case["kind"] == "reload":     # rows in, rows stored, rows read, rows out
        return {"bytes": 4 * 2 * ROW * sum(_histories(case)) * L, "flops": 0}
    items = _items(case)
    n = sum(it[2] for it in items)
    live = sum(it[1] for it in items)
    used = {it[0] for it in items if it[0] >= 0}
    live += len(used) * case["prefix_len"]
    rows = live + 2 * n
    if case["kind"] == "start":      # the observation's rows come in and are stored first
        rows += 2 * case["prefix_len"]
    bytes_ = rows * 2 * ROW + n * HEADS * 2 * ROW + (n * HEADS * 4 if case["lse"] else 0)
    return {"bytes": bytes_ * L, "flops": _visible(case) * HEADS * 4 * DIM * L}


def tolerance(case):
    """Outputs are rounded to bf16 and split results to 16 bits with a scale per row: against
    64 bits the relative error is 1.7e-3, the largest single one 4.6e-3 of the rms.  Loaded rows
    come back as they went in."""
    if case["kind"] == "reload":
        return "exact"
    return {"rel": 7e-3, "max": 2e-2}


def exact(case, seed):
    """Softmax attention of every item over its own visible set, in 64 bits."""
    L = case["layers"]
    if case["kind"] == "reload":
        return {"kv": torch.stack([_history_rows(case, seed, l) for l in range(L)]).double()}
    outs, lses = [], []
    for l in range(L):
        pre = [_prefix_rows(case, seed, i, l).double() for i in range(case["prefixes"])]
        hist = _history_rows(case, seed, l).double() if case["decoders"] else None
        new, q = _step_rows(case, seed, l)
        new, q = new.double(), q.double()
        o, z = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float64, device="cuda")
        t = at = 0
        for p, h, n, both in _items(case):
            parts = [pre[p]] if p >= 0 else []
            if h:
                parts.append(hist[:, at:at + h])
                at += h
            k, v = torch.cat(parts + [new[:, t:t + n]], dim=1)
            logits = (q[t:t + n].reshape(n * HEADS, DIM) @ k.t()).view(n, HEADS, -1) * SCALE
            if not both:
                last = k.shape[0] - n + torch.arange(n, device="cuda")   # own position
                hidden = torch.arange(k.shape[0], device="cuda") > last[:, None]
                logits = logits.masked_fill(hidden[:, None, :], -math.inf)
            z[t:t + n] = torch.logsumexp(logits, dim=2)
            o[t:t + n] = (torch.softmax(logits, dim=2).view(n * HEADS, -1) @ v).view(n, HEADS, DIM)
            t += n
        outs.append(o)
        lses.append(z)
    got = {"out": torch.stack(outs)}
    if case["lse"]:
        got["lse"] = torch.stack(lses)
    return got
