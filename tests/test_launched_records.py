"""The records that a launch reads, on host-only pools (no GPU): every (query, key) pair lies in exactly one
of them, also where two share an item; inline token and block ids; the flag of the page loads."""
import numpy as np
import pytest

from paper_2603_14371_amd import binding as B

NO_CAUSAL = 0x3fffffff
PATH_MASK, FRESH, APPENDS, ONCE, ROW_SHIFT = 15, 16, 32, 64, 8


class _Pool:
    def __init__(self, num_blocks=8192, n_layers=1, **kw):
        order = np.random.default_rng(5).permutation(num_blocks).astype(np.int32)
        self.h = B.oxy_pool_create(B.make_config(
            n_layers, num_blocks, free_order=order, flags=B.POOL_HOST_ONLY, max_partials=1 << 16,
            max_q_tokens=2048, max_append_tokens=1 << 16, **kw))

    def prefix(self, n):
        pid = B.oxy_prefix_create(self.h)
        if n:
            B.oxy_prefix_append(self.h, pid, 0, 0, 0, n, 0, 0)
        return pid

    def stream(self, pid, kind, hist=0):
        sid = B.oxy_stream_create(self.h, pid, kind)
        if hist:
            B.oxy_batch_destroy(B.oxy_batch_build(self.h, [(sid, hist)], B.BATCH_APPEND_ONLY, 0))
        return sid

    def build(self, items):
        """The batch's launched records without padding, checked; its work items; its info."""
        self.before = [B.oxy_stream_info(self.h, sid) for sid, _ in items]
        batch = B.oxy_batch_build(self.h, items, 0, 0)
        rec, work, info = B.oxy_batch_records(batch), B.oxy_batch_work(batch), B.oxy_batch_info(batch)
        B.oxy_batch_destroy(batch)
        self.launched = rec
        rec, work = rec[rec[:, 7] & PATH_MASK != 2], work[work[:, 7] != 2]
        self._check(items, rec, info)
        return rec, work, info

    def _check(self, items, rec, info):
        tok = []   # of every query token: item, prefix blocks, own blocks, prefix keys, own keys
        for i, ((sid, n), (pid, kind, old, _)) in enumerate(zip(items, self.before)):
            old = old if kind == B.KIND_DECODE else 0
            pre = (B.oxy_prefix_blocks(self.h, pid), B.oxy_prefix_info(self.h, pid)[0]) if pid >= 0 else ([], 0)
            own = B.oxy_stream_blocks(self.h, sid)
            for t in range(n):
                tok.append((i, pre[0], own, pre[1], old + t + 1 if kind == B.KIND_DECODE else n, old + t))
        keys = [[] for _ in tok]   # (phase, begin, end) per token
        parts = [[] for _ in tok]
        for r in rec:
            n, lo, hi, q0, part = (int(r[c]) for c in (1, 3, 4, 5, 6))
            assert 1 <= n <= 8 and 0 <= lo < hi and lo % 32 == 0
            assert np.all(r[8 + n:16] == r[8 + n - 1])                       # inline ids: the last repeated
            pages = r[16:32].tolist()
            for k in range(n):
                t = int(r[8 + k])
                i, pre, own, n_pre, n_own, pos = tok[t]
                src = own if pages[0] in own else pre
                want = src[lo // 16:-(-hi // 16)][:16]
                assert pages == want + want[-1:] * (16 - len(want))
                end = hi
                if q0 != NO_CAUSAL:
                    assert src is own and pos == q0 + k                      # the causal base is the first token's
                    end = min(hi, pos + 1)
                if lo < end:
                    keys[t].append((src is own, lo, end))
                parts[t].append(part)
                if int(r[7]) & FRESH:
                    assert src is own and self.before[i][1:3] != (B.KIND_DECODE, 1)
                    first = int(r[7]) >> ROW_SHIFT                           # the item's first token of the step
                    assert tok[first][0] == i and (first == 0 or tok[first - 1][0] != i)
        for t, (i, pre, own, n_pre, n_own, pos) in enumerate(tok):
            assert sorted(parts[t]) == list(range(len(parts[t]))), "token %d" % t
            for phase, n_keys in ((False, n_pre), (True, n_own)):
                spans = sorted(s[1:] for s in keys[t] if s[0] == phase)
                assert [s[0] for s in spans] + [n_keys] == [0] * (n_keys > 0) + [s[1] for s in spans] \
                    or (n_keys == 0 and not spans), "token %d" % t
        assert sum(len(p) for p in parts) == info[3]

    def close(self):
        B.oxy_pool_destroy(self.h)


@pytest.mark.parametrize("kind", [B.KIND_ACTION, B.KIND_DECODE], ids=["bidirectional", "causal"])
@pytest.mark.parametrize("chunk", [3, 4, 5, 6, 8, 9, 12, 13, 32, 33, 37, 50, 62, 64])
@pytest.mark.parametrize("prefix_len", [0, 64, 832])
def test_two_records_share_an_item_of_a_short_chunk_in_a_small_launch(prefix_len, chunk, kind):
    p = _Pool()
    pid = p.prefix(prefix_len)
    rec, work, info = p.build([(p.stream(pid, B.KIND_DECODE, 40), 1), (p.stream(pid, kind), chunk)])
    p.close()
    wide = work[(work[:, 7] == 1) & (work[:, 1] > 4)]
    fits = len(work) + len(wide) <= 256
    assert fits or (prefix_len == 832 and chunk >= 62)
    assert len(rec) == len(work) + (len(wide) if fits else 0) and info[2] >= len(work)
    # of every such item: two records that follow each other in tokens and causal base, all else alike
    for w in wide:
        mine = [r for r in rec if w[0] <= r[0] < w[0] + w[1] and np.array_equal(r[[2, 3, 4, 6]], w[[2, 3, 4, 6]])]
        mine.sort(key=lambda r: r[0])
        if not fits:
            assert len(mine) == 1 and mine[0][1] == w[1]
            continue
        a, b = mine
        assert a[0] == w[0] and a[1] == 4 and b[0] == w[0] + 4 and b[1] == w[1] - 4
        assert a[5] == w[5] and b[5] == (w[5] if w[5] == NO_CAUSAL else w[5] + 4)
        assert a[7] == b[7] and a[7] & FRESH and a[7] & PATH_MASK == w[7]


def test_items_are_shared_up_to_256_workgroups_and_within_the_limit():
    """Further requests take the launch past 256 records, or the pool's own limit does."""
    seen = set()
    for n_req in range(0, 40, 3):
        p = _Pool()
        pid = p.prefix(832)
        items = [(p.stream(pid, B.KIND_ACTION), 50)] + [(p.stream(pid, B.KIND_DECODE), 1) for _ in range(n_req)]
        rec, work, _ = p.build(items)
        p.close()
        wide = int(((work[:, 7] == 1) & (work[:, 1] > 4) & (work[:, 4] <= 50)).sum())
        assert len(rec) - len(work) == (wide if len(work) + wide <= 256 else 0)
        seen.add(len(rec) > len(work))
        if len(rec) > len(work):
            for room, shared in ((len(rec), True), (len(rec) - 1, False)):
                p = _Pool(max_work_items=room)
                pid = p.prefix(832)
                items = [(p.stream(pid, B.KIND_ACTION), 50)] + \
                    [(p.stream(pid, B.KIND_DECODE), 1) for _ in range(n_req)]
                r, w, _ = p.build(items)
                p.close()
                assert len(w) == len(work) and (len(r) > len(w)) == shared
    assert seen == {True, False}


@pytest.mark.parametrize("n,prefix_len,chunk,shares", [
    (6, 1500, 50, True), (7, 832, 50, True), (6, 2048, 50, True), (7, 832, 47, True), (5, 832, 50, False),
    (8, 832, 50, False), (8, 1000, 50, False), (1, 832, 400, False)])
def test_chunks_alone_share_items_beyond_one_for_each_cu(n, prefix_len, chunk, shares):
    """Items of more than four tokens on prefix pages, more than 256 of them and slots left: some are two
    records of at most four, while all such have a slot; beside a request none is."""
    def launch(request=False):
        p = _Pool()
        pids = [p.prefix(prefix_len) for _ in range(n)]
        items = [(p.stream(pid, B.KIND_ACTION), chunk) for pid in pids]
        items += [(p.stream(pids[0], B.KIND_DECODE, 5), 1)] if request else []
        out = p.build(items)
        p.close()
        return out[0], out[1]
    rec, work = launch()
    assert (len(rec) > len(work)) == shares
    if shares:
        assert len(rec) <= 512
        where = lambda r, d=0: (r[0] - d, *r[[2, 3, 4, 6]])   # noqa: E731
        first, listed = {where(r): r[1] for r in rec}, {where(r) for r in work}
        second = [r for r in rec if where(r) not in listed]
        assert len(second) == len(rec) - len(work)
        assert all(1 <= r[1] <= 4 and first[where(r, 4)] == 4 for r in second)
        mixed, listed = launch(request=True)
        assert len(mixed) == len(listed)


@pytest.mark.parametrize("n,prefix_len,hist,n_new", [
    (3, 0, 1700, 100), (3, 64, 1700, 100), (3, 0, 1700, 101), (5, 64, 1500, 53), (4, 832, 1500, 50)])
def test_causal_items_on_long_histories_are_shared_too(n, prefix_len, hist, n_new):
    """Several new tokens behind a long history: of a shared item the second record's causal base is four further on,
    and the first one keeps the keys of both."""
    p = _Pool()
    pid = p.prefix(prefix_len) if prefix_len else -1
    rec, work, _ = p.build([(p.stream(pid, B.KIND_DECODE, hist + 7 * i), n_new) for i in range(n)])
    p.close()
    listed = {tuple(w[[0, 2, 3, 4, 6]]): w for w in work}
    second = [r for r in rec if tuple(r[[0, 2, 3, 4, 6]]) not in listed]
    assert second and len(second) == len(rec) - len(work)
    for r in second:
        at = (r[0] - 4, *r[[2, 3, 4, 6]])
        first = [f for f in rec if tuple(f[[0, 2, 3, 4, 6]]) == at]
        assert len(first) == 1 and first[0][1] == 4 and r[1] == listed[at][1] - 4 and r[7] == first[0][7]
        assert r[5] == (NO_CAUSAL if first[0][5] == NO_CAUSAL else first[0][5] + 4)
    assert any(r[5] != NO_CAUSAL for r in second)


def _by_size(records):
    """The records of every XCD in the order of their size: of more than 32, the largest of the first 32 is
    dealt out with the smallest of the next 32."""
    for x in range(8):
        q = [r for r in records[x::8] if r[7] & PATH_MASK != 2]
        if len(q) > 32:
            top = min(len(q), 64)
            m, r = top - 32, [None] * top
            for j in range(m):
                r[32 - m + j], r[top - 1 - j] = q[j], q[32 + j]
            for j in range(m, 32):
                r[j - m] = q[j]
            q[:top] = r
        yield q


@pytest.mark.parametrize("n,prefix_len,chunk", [
    (7, 832, 45), (7, 832, 46), (7, 832, 47), (7, 832, 53), (6, 1500, 45), (6, 1500, 50), (6, 2048, 53)])
def test_halved_items_are_ordered_by_the_tokens_each_record_has(n, prefix_len, chunk):
    """An XCD's records of three and four tokens on a whole split of a prefix stand together in the order of
    size, behind those of more tokens: also the ones whose item has one or two tokens left for the other record."""
    p = _Pool()
    rec, work, _ = p.build([(p.stream(p.prefix(prefix_len), B.KIND_ACTION), chunk) for _ in range(n)])
    p.close()
    assert len(rec) > len(work)
    halved = 0
    for q in _by_size(p.launched):
        most = max(r[4] - r[3] for r in q)
        kind = [0 if r[4] - r[3] < most else 2 if r[1] > 4 else int(r[1] > 2) for r in q]   # 0: all others
        kind = "".join(str(k) for k in kind)
        assert kind == "2" * kind.count("2") + kind.lstrip("2") and "1" * kind.count("1") in kind
        halved += kind.count("1")
    assert halved


@pytest.mark.parametrize("seed", range(30))
def test_every_pair_of_query_and_key_in_one_record(seed):
    rng = np.random.default_rng(8000 + seed)
    p = _Pool()
    pids = [p.prefix(int(rng.choice([0, 17, 64, 190, 832, 1100, 2048]))) for _ in range(int(rng.integers(1, 5)))]
    items = [(p.stream(int(rng.choice(pids)), B.KIND_DECODE, int(rng.choice([0, 1, 30, 200, 600, 1500]))),
              int(rng.choice([1, 1, 2, 3, 5, 13, 64, 70]))) for _ in range(int(rng.integers(0, 9)))]
    items += [(p.stream(int(rng.choice(pids)), B.KIND_ACTION), int(rng.integers(1, 130)))
              for _ in range(int(rng.integers(1, 4)))]
    p.build([items[i] for i in rng.permutation(len(items))])
    p.close()


def test_pages_are_loaded_past_the_caches_above_128_mb():
    """2048 live tokens are 2 MB in a layer: own pages of decode items only, from the 65th layer on."""
    for n_layers, once in ((1, False), (64, False), (65, True)):
        p = _Pool(n_layers=n_layers)
        pid = p.prefix(1024)
        rec, _, _ = p.build([(p.stream(pid, B.KIND_DECODE, 972), 2), (p.stream(pid, B.KIND_ACTION), 50)])
        p.close()
        own = rec[rec[:, 7] & APPENDS != 0]
        assert len(own) == 4 and np.all((own[:, 7] & ONCE != 0) == once)
        assert not np.any(rec[rec[:, 7] & APPENDS == 0][:, 7] & ONCE)
