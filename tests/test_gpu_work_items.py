"""Work items at the sizes where their tiling can go wrong: key ranges around one 32-key step, one
round of 128 keys and several rounds, one to nine query tokens per item, both append forms; the
softmax scale's sign and zero; values far from magnitude one."""
import numpy as np
import pytest

from paper_2603_14371_amd import synth
from paper_2603_14371_amd.synth import ACTION, DECODE, _TraceBuilder, _workload
from parity_util import run_both

pytestmark = pytest.mark.gpu


def _step(prefix_len, chunk, hist, n_new, n_layers=1):
    b = _TraceBuilder()
    pid = b.prefix(prefix_len)
    act, dec = b.stream(pid, ACTION), b.stream(pid, DECODE)
    if hist:
        b.step([(dec, hist)], attend=False)
    b.step([(act, chunk), (dec, n_new)])
    return _workload("work_items", 5150, n_layers, 512, b.trace)


# the tolerance is the suite's own (bf16 outputs, see parity_util)
@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
@pytest.mark.parametrize("prefix_len,chunk,hist,n_new,split", [
    (1, 1, 0, 1, 0), (31, 3, 31, 1, 0), (33, 4, 126, 2, 0), (127, 5, 127, 2, 128),
    (128, 6, 128, 1, 128), (129, 7, 255, 2, 256), (160, 8, 256, 1, 256), (383, 9, 383, 3, 384),
    (385, 2, 384, 8, 384), (1025, 9, 513, 9, 0), (2048, 65, 1023, 1, 1024), (1040, 130, 40, 5, 512),
])
def test_edges_of_steps_rounds_and_tiles(prefix_len, chunk, hist, n_new, split, fold):
    w = _step(prefix_len, chunk, hist, n_new)
    gw, _, _, _ = run_both(w, poison=True, split_tokens=split, stream_split_tokens=split,
                           max_partials=8192, fold_append=fold)
    gw.close()


@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
@pytest.mark.parametrize("prefix_len", [34, 63, 64, 65, 191, 192])
@pytest.mark.parametrize("chunk,hist,n_new", [(1, 60, 4), (4, 29, 3), (2, 70, 1)])
def test_splits_of_at_most_64_keys(prefix_len, chunk, hist, n_new, fold):
    """Two of the four wavefronts have no keys there: they load none and add nothing."""
    gw, _, _, _ = run_both(_step(prefix_len, chunk, hist, n_new), poison=True, fold_append=fold)
    gw.close()


@pytest.mark.parametrize("scale", [-1.0 / 16, 0.0])
def test_softmax_scale_may_be_negative_or_zero(scale):
    w = _step(150, 9, 140, 1)
    w["scale"] = scale
    gw, _, _, _ = run_both(w, poison=True, fold_append=True)
    gw.close()


@pytest.mark.parametrize("power", [-60, 60])
def test_magnitude_of_the_values_does_not_enter_the_rounding(power):
    """Values times a power of two give exactly the outputs times that power: split results carry
    their own exponents (all intermediate values stay normal at these powers)."""
    from paper_2603_14371_amd.harness import GpuWorld
    w = _step(300, 9, 140, 1)
    src = synth.DataSource(w["seed"])

    def scaled(recipe, layer, what, n):
        bits = src(recipe, layer, what, n)
        if what != "v":
            return bits
        return np.where((bits & 0x7F80) != 0, bits + np.int32(power * 128), bits).astype(np.uint16)
    outs = []
    for data in (src, scaled):
        gw = GpuWorld(w, data, poison=True)
        outs.append(gw.run(w["trace"])[-1]["O"][0].astype(np.int32))
        gw.close()
    nonzero = (outs[0] & 0x7F80) != 0
    assert nonzero.mean() > 0.99
    assert np.array_equal(outs[0][nonzero] + power * 128, outs[1][nonzero])


@pytest.mark.parametrize("n,prefix_len,chunk", [(7, 832, 50), (6, 1500, 47)])
@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
def test_items_of_chunks_that_two_records_share_equal_the_chunk_alone(n, prefix_len, chunk, fold):
    from paper_2603_14371_amd.harness import GpuWorld
    b = _TraceBuilder()
    acts = [b.stream(b.prefix(prefix_len), ACTION) for _ in range(n)]
    w = _workload("shared_items", 5153, 1, 1024, b.trace)
    gw = GpuWorld(w, synth.DataSource(w["seed"]), max_q_tokens=512, max_append_tokens=512, max_partials=16384,
                  fold_append=fold, poison=True)
    gw.run(w["trace"])
    data = {"tag": 901, "tok0": 0, "n_total": n * chunk}
    alone = [gw.step({"op": "step", "items": [(a, chunk)], "data": dict(data, tok0=i * chunk)})
             for i, a in enumerate(acts)]
    whole = gw.step({"op": "step", "items": [(a, chunk) for a in acts], "data": data})
    gw.close()
    for key in ("O", "LSE"):
        assert np.array_equal(whole[key][0], np.concatenate([r[key][0] for r in alone]))


@pytest.mark.parametrize("n,prefix_len,hist,n_new", [(3, 64, 1700, 100), (5, 64, 1500, 53)])
def test_causal_items_that_two_records_share_equal_the_request_alone(n, prefix_len, hist, n_new):
    """Several new tokens behind long histories, some splits past the diagonal of an item's first four tokens:
    the oracle's values, and the bits of each request by itself."""
    b = _TraceBuilder()
    sids = [b.stream(b.prefix(prefix_len), DECODE) for _ in range(n)]
    b.step([(s, hist + 7 * i) for i, s in enumerate(sids)], attend=False)
    b.step([(s, n_new) for s in sids], recipe=b.recipe(n * n_new, tag=902))
    w = _workload("shared_causal_items", 5154, 1, 1024, b.trace)
    gw, res, _, _ = run_both(w, poison=True, max_q_tokens=512, max_partials=16384)
    for i, s in enumerate(sids):
        gw.apply({"op": "stream_rewind", "sid": s, "len": hist + 7 * i})
    alone = [gw.step({"op": "step", "items": [(s, n_new)], "data": {"tag": 902, "tok0": i * n_new, "n_total": n * n_new}})
             for i, s in enumerate(sids)]
    gw.close()
    for key in ("O", "LSE"):
        assert np.array_equal(res[-1][key][0], np.concatenate([r[key][0] for r in alone]))


@pytest.mark.parametrize("n_prefix,prefix_len,width", [(3, 832, 4), (9, 832, 8), (9, 190, 4)])
@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
def test_items_in_a_launch_of_many_equal_items_alone(n_prefix, prefix_len, width, fold):
    """A launch of many work items stacks a short prefix's queries in wider items; every query's
    bits are those of its item in a batch of its own."""
    from paper_2603_14371_amd import binding as B
    from paper_2603_14371_amd.harness import GpuWorld
    b = _TraceBuilder()
    pids = [b.prefix(prefix_len) for _ in range(n_prefix)]
    acts = [b.stream(p, ACTION) for p in pids]
    decs = [b.stream(pids[i % 2], DECODE) for i in range(5)]
    b.step([(d, 20 + 31 * i) for i, d in enumerate(decs)], attend=False)
    items = [(a, 50) for a in acts] + [(d, 1 + i % 2) for i, d in enumerate(decs)]
    n_tok = sum(n for _, n in items)
    w = _workload("many_items", 5152, 1, 1024, b.trace)
    gw = GpuWorld(w, synth.DataSource(w["seed"]), max_q_tokens=512, max_append_tokens=512,
                  max_partials=16384, fold_append=fold, poison=True)
    gw.run(w["trace"])
    data = {"tag": 900, "tok0": 0, "n_total": n_tok}
    alone, t0 = [], 0
    for sid, n in items:
        r = gw.step({"op": "step", "items": [(sid, n)], "data": dict(data, tok0=t0)})
        alone.append((r["O"][0], r["LSE"][0]))
        if sid in decs:
            B.oxy_stream_rewind(gw.pool, sid, B.oxy_stream_info(gw.pool, sid)[2] - n)
        t0 += n
    batch = B.oxy_batch_build(gw.pool, items, 0, gw._stream())
    work = B.oxy_batch_work(batch)
    B.oxy_batch_destroy(batch)
    for sid, n in items:
        if sid in decs:
            B.oxy_stream_rewind(gw.pool, sid, B.oxy_stream_info(gw.pool, sid)[2] - n)
    prefix_phase = work[(work[:, 5] == 0x3fffffff) & (work[:, 4] > 50)]
    assert set(int(x) for x in prefix_phase[:, 1]) >= {width}
    assert int(prefix_phase[:, 1].max()) == width
    r = gw.step({"op": "step", "items": items, "data": data})
    gw.close()
    assert np.array_equal(np.concatenate([o for o, _ in alone]), r["O"][0])
    assert np.array_equal(np.concatenate([l for _, l in alone]), r["LSE"][0])


@pytest.mark.parametrize("n,prefix_len,hist,n_new", [(3, 64, 1700, 100), (5, 64, 1500, 53)])
def test_causal_items_that_two_records_share_equal_the_request_alone(n, prefix_len, hist, n_new):
    """Several new tokens behind long histories, some splits past the diagonal of an item's first four tokens:
    the oracle's values, and the bits of each request by itself."""
    b = _TraceBuilder()
    sids = [b.stream(b.prefix(prefix_len), DECODE) for _ in range(n)]
    b.step([(s, hist + 7 * i) for i, s in enumerate(sids)], attend=False)
    b.step([(s, n_new) for s in sids], recipe=b.recipe(n * n_new, tag=902))
    w = _workload("shared_causal_items", 5154, 1, 1024, b.trace)
    gw, res, _, _ = run_both(w, poison=True, max_q_tokens=512, max_partials=16384)
    for i, s in enumerate(sids):
        gw.apply({"op": "stream_rewind", "sid": s, "len": hist + 7 * i})
    alone = [gw.step({"op": "step", "items": [(s, n_new)], "data": {"tag": 902, "tok0": i * n_new, "n_total": n * n_new}})
             for i, s in enumerate(sids)]
    gw.close()
    for key in ("O", "LSE"):
        assert np.array_equal(res[-1][key][0], np.concatenate([r[key][0] for r in alone]))


@pytest.mark.parametrize("n_prefix,prefix_len,width", [(2, 1100, 4), (3, 2048, 4), (9, 1300, 8)])
@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
def test_the_same_on_long_prefixes(n_prefix, prefix_len, width, fold):
    """The same rule on prefixes whose splits take two rounds of 128 keys, the second one partly."""
    test_items_in_a_launch_of_many_equal_items_alone(n_prefix, prefix_len, width, fold)


@pytest.mark.parametrize("pick", ["in_order", "reversed", "every_third", "repeated", "shuffled"])
def test_gather_of_any_slot_list(pick):
    """Read-back accepts slots in any order and any number of times: whole blocks, parts of a block
    and single tokens, more runs than one launch carries."""
    from paper_2603_14371_amd.harness import GpuWorld
    b = _TraceBuilder()
    dec = b.stream(-1, DECODE)
    op = b.step([(dec, 611)], attend=False)
    w = _workload("gather", 5153, 1, 64, b.trace, free_order=np.random.default_rng(3).permutation(64))
    src = synth.DataSource(w["seed"])
    gw = GpuWorld(w, src, poison=True)
    gw.run(w["trace"])
    k, v = (src(op["data"], 0, what, 611) for what in "kv")
    n = np.arange(611)
    order = {"in_order": n, "reversed": n[::-1], "every_third": n[5::3], "repeated": np.repeat(n, 2),
             "shuffled": np.random.default_rng(4).permutation(611)}[pick]
    slots = gw.stream_slots(dec)
    gk, gv = gw.gather(0, [slots[i] for i in order])
    gw.close()
    assert np.array_equal(gk, k[order]) and np.array_equal(gv, v[order])


def _launched(prefix_len, chunk, decoders, n_layers=1):
    """Records (padding left out), work items and split results of a step of one chunk and
    `decoders` = (own history, new tokens) each, all on one prefix; from a host-only pool."""
    from paper_2603_14371_amd import binding as B
    pool = B.oxy_pool_create(B.make_config(n_layers, 4096, flags=B.POOL_HOST_ONLY, max_q_tokens=512,
                                           max_append_tokens=1 << 16, max_partials=8192))
    pid = B.oxy_prefix_create(pool)
    B.oxy_prefix_append(pool, pid, 0, 0, 0, prefix_len, 0, 0)
    items = [(B.oxy_stream_create(pool, pid, B.KIND_ACTION), chunk)]
    for hist, n_new in decoders:
        items.append((B.oxy_stream_create(pool, pid, B.KIND_DECODE), n_new))
        if hist:
            B.oxy_batch_destroy(B.oxy_batch_build(pool, [(items[-1][0], hist)], B.BATCH_APPEND_ONLY, 0))
    batch = B.oxy_batch_build(pool, items, 0, 0)
    rec, work, n_partials = B.oxy_batch_records(batch), B.oxy_batch_work(batch), B.oxy_batch_info(batch)[3]
    B.oxy_batch_destroy(batch)
    B.oxy_pool_destroy(pool)
    return rec[rec[:, 7] & 15 != 2], work[work[:, 7] != 2], n_partials


@pytest.mark.parametrize("hist,n_new", [(40, 1), (127, 2), (300, 1), (520, 2)])
def test_own_pages_read_past_the_caches_give_the_same_bits(hist, n_new):
    """The non-temporal loads are taken where the pages of all layers are more than 128 MB: the same
    layer in a pool of one layer and in one of enough layers, written and read by the work items."""
    outs, marked = [], []
    for n_layers in (1, 1 + (128 << 20) // ((300 + hist) << 10)):
        w = _step(300, 9, hist, n_new, n_layers)
        w["num_blocks"] = 64
        rec, _, _ = _launched(300, 9, [(hist, n_new)], n_layers)
        own = rec[rec[:, 7] & 32 != 0]             # a decode item's own pages; 64 = past the caches
        marked.append(set((own[:, 7] & 64).tolist()))
        gw, g, _, _ = run_both(w, layers=[0], poison=True, fold_append=True)
        outs.append(g[-1])
        gw.close()
    assert marked == [{0}, {64}]
    assert np.array_equal(outs[0]["O"][0], outs[1]["O"][0])
    assert np.array_equal(outs[0]["LSE"][0], outs[1]["LSE"][0])


@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
@pytest.mark.parametrize("prefix_len,chunk", [(256, n) for n in (3, 5, 8, 12, 32, 33, 62, 64)] + [(832, 62), (832, 64)])
def test_width_of_a_short_chunks_own_tiles(prefix_len, chunk, fold):
    """A chunk's tiles shared by two workgroups in a small launch and whole in one of more than 256, and their
    split results left in the caches and written through (more than 1280 of them there, 640 in a launch
    of at most 256): the same bits, and the oracle's values.  On 832 tokens a long chunk alone has whole
    tiles, beside 40 requests (whose prefix items are wider) shared ones."""
    if prefix_len == 256:   # (requests, tiles shared, written through)
        batches = [(1, chunk > 4, False), (50 if chunk <= 33 else 24, False, False), (260, False, True)]
    else:
        batches = [(1, False, False), (40, True, True)]
    outs = []
    for n_dec, shared, through in batches:
        rec, work, n_partials = _launched(prefix_len, chunk, [(0, 1)] * n_dec)
        assert (len(rec) > len(work)) == shared
        assert (n_partials > (640 if len(rec) <= 256 else 1280)) == through
        b = _TraceBuilder()
        pid = b.prefix(prefix_len)
        act = b.stream(pid, ACTION)
        dec = [b.stream(pid, DECODE) for _ in range(n_dec)]
        b.step([(act, chunk)] + [(d, 1) for d in dec])
        w = _workload("short_tiles", 5151, 1, 512, b.trace)
        gw, g, _, _ = run_both(w, poison=True, fold_append=fold, max_q_tokens=512, max_append_tokens=512)
        outs.append(g[-1])
        gw.close()
    for o in outs[1:]:
        assert np.array_equal(outs[0]["O"][0][:chunk], o["O"][0][:chunk])
        assert np.array_equal(outs[0]["LSE"][0][:chunk], o["LSE"][0][:chunk])


@pytest.mark.parametrize("first,then", [(1, 3), (4, 4), (7, 2), (8, 8), (11, 5), (12, 20), (15, 1), (17, 14)])
def test_parts_of_a_block_leave_its_other_rows(first, then):
    """A block's rows written in two parts that meet inside a V chunk, at its end and at a block's end, then
    a range across the seam written again; and chunks of the same lengths on an empty history,
    whose rows the merge launch writes.  Pool contents bit for bit."""
    from parity_util import assert_pool_contents_equal
    b = _TraceBuilder()
    pid = b.prefix(first)
    b.trace.append({"op": "prefix_append", "pid": pid, "n": then, "pos0": first, "data": b.recipe(then)})
    if first > 1:
        b.trace.append({"op": "prefix_append", "pid": pid, "n": 2, "pos0": first - 1, "data": b.recipe(2)})
    acts = [b.stream(pid, ACTION) for _ in range(2)]
    b.step([(acts[0], first + then), (acts[1], first + 2)])
    w = _workload("parts", 5154, 2, 64, b.trace)
    gw, _, ow, _ = run_both(w, poison=True, fold_append=True)
    n = assert_pool_contents_equal(gw, ow)
    gw.close()
    assert n == 2 * (2 * (first + then) + first + 2)
