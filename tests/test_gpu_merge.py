"""The merge of a token's split results at the counts where its form changes: up to 4, 8, 12 and 16
at once, sixteen at a time beyond; tokens of different counts beside each other."""
import pytest

from paper_2603_14371_amd.synth import ACTION, DECODE, _TraceBuilder, _workload
from parity_util import run_both

pytestmark = pytest.mark.gpu


# the tolerance is the suite's own (bf16 outputs, see parity_util)
@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
@pytest.mark.parametrize("counts", [[1], [4], [5], [16], [17], [33], [12, 13, 3], [8, 9, 1, 32],
                                    [2, 15, 7, 31, 11, 48, 6, 10, 14]], ids=str)
def test_split_results_of_a_token(counts, fold):
    """Decode streams without a prefix: a history of 32 n tokens is n split results of 32 keys.  The
    chunk beside them has its own count (prefix and own tokens)."""
    _compare(counts, 5, fold)


@pytest.mark.parametrize("fold", [False, True], ids=["separate_append", "folded_append"])
@pytest.mark.parametrize("counts", [[4, 5, 8, 9, 12, 13], [16, 17, 33, 15, 14, 1, 48]], ids=str)
def test_split_results_of_a_token_among_many(counts, fold):
    """The same in a launch of more than 256 tokens, whose merge workgroups take all heads of a token."""
    _compare(counts, 260, fold)


def _compare(counts, chunk, fold):
    b = _TraceBuilder()
    act = b.stream(b.prefix(70), ACTION)
    streams = [b.stream(-1, DECODE) for _ in counts]
    hist = [(s, 32 * n - 1) for s, n in zip(streams, counts)]
    b.step([h for h in hist if h[1]], attend=False)
    b.step([(s, 1) for s in streams] + [(act, chunk)])
    w = _workload("merge", 5160, 1, 1024, b.trace)
    gw, _, _, _ = run_both(w, poison=True, split_tokens=32, stream_split_tokens=32, max_partials=8192,
                           fold_append=fold)
    gw.close()
