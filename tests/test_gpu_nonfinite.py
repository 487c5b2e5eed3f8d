"""A value that is not finite gives no wrong finite output.  Output dimensions are independent sums; split
results hold 64 of them under one exponent, so an infinite sum may take its 64 along as NaN, and all
others equal the oracle's for the same inputs without it."""
import numpy as np
import pytest

from oracle import attention
from oracle.replay import OracleWorld
from paper_2603_14371_amd import synth
from paper_2603_14371_amd.synth import ACTION, DECODE, _TraceBuilder, _workload
from parity_util import assert_lse_close, assert_o_close

pytestmark = pytest.mark.gpu

INF, NAN = 0x7F80, 0x7FC0


@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
@pytest.mark.parametrize("bits", [INF, INF | 0x8000, NAN], ids=["inf", "-inf", "nan"])
@pytest.mark.parametrize("where", ["prefix", "chunk", "history"])
@pytest.mark.parametrize("n_prefix", [1, 12])
def test_a_value_that_is_not_finite_gives_no_wrong_finite_output(where, bits, fold, n_prefix):
    from paper_2603_14371_amd.harness import GpuWorld
    b = _TraceBuilder()
    pids = [b.prefix(300, b.recipe(300, tag=100 + i)) for i in range(n_prefix)]
    acts = [b.stream(p, ACTION) for p in pids]
    dec = b.stream(pids[0], DECODE)
    b.tag = 10
    b.step([(dec, 150)], attend=False)                              # tag 10
    b.step([(a, 50) for a in acts] + [(dec, 1)])                    # tag 11
    w = _workload("nonfinite", 5180, 1, 512, b.trace)
    src = synth.DataSource(w["seed"])
    at = {"prefix": (100, 17), "chunk": (11, 9), "history": (10, 70)}[where]
    dim = 133

    def planted(recipe, layer, what, n):
        x = src(recipe, layer, what, n)
        if what == "v" and recipe["tag"] == at[0]:
            x = x.copy()
            x[at[1] - recipe["tok0"], dim] = bits
        return x

    gw = GpuWorld(w, planted, poison=True, fold_append=fold)
    ow = OracleWorld(w["num_blocks"], 1, src, w["scale"])
    for op in w["trace"]:
        g, o = gw.apply(op), ow.apply(op)
    gw.close()
    got, ref = g["O"][0], o["O"][0]
    sees = {"prefix": list(range(50)) + [len(ref) - 1], "chunk": list(range(50)),
            "history": [len(ref) - 1]}[where]
    assert not np.isfinite(attention.widen_bf16(got[sees][:, :, dim])).any()
    part = np.arange(256) // 64 == dim // 64
    assert_o_close(got[:, :, ~part], ref[:, :, ~part], where)
    lost = ~np.isfinite(attention.widen_bf16(got[:, :, part]))
    assert np.all(lost.all(axis=2) | (lost.sum(axis=2) <= 1))     # the 64 dims, or the value's own
    assert_o_close(got[:, :, part][~lost], ref[:, :, part][~lost], where)
    rest = np.setdiff1d(np.arange(len(ref)), sees)
    if len(rest):
        assert_o_close(got[rest], ref[rest], where)
    assert_lse_close(g["LSE"][0], o["LSE"][0], where)
