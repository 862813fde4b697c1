"""The encoder's attention where its two splits of the work begin and end, on
the GPU against the oracle (helpers and tolerance of test_gpu_encoder.py).

A sequence of few rows gives each wave a share of the keys (four waves to 32
queries, 64 queries a workgroup); a longer one gives each wave 32 queries of its
own (128 a workgroup, 64-key tiles).  Sequence lengths sit at and beside
multiples of the 32-key blocks, the 64- and 128-key tiles and the 32-, 64- and
128-query blocks, so tiles end in masked keys, waves have no keys or no
queries, and steps straddle the diagonal.  At d = 512 (four heads) sequences of
up to 2048 rows (3072 when causal) are of the first kind, at d = 2048 of up to
512 (768).
"""
import numpy as np
import pytest

from tests.test_gpu_encoder import _case, _check, _oracle, _run

pytestmark = pytest.mark.gpu

EDGES = (1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160, 193)      # rows a sequence, text included
D = 512


def _split_edges(lengths):
    texts = [min(7, n - 1) for n in lengths]
    return [n - t for n, t in zip(lengths, texts)], texts


@pytest.mark.parametrize("causal", [False, True], ids=["bidirectional", "causal"])
@pytest.mark.parametrize("extra", [0, 1, 2400], ids=["few_rows", "over_the_edge", "many_rows"])
def test_attention_splits(gpu_lib, extra, causal):
    # short sequences in batches of few and of many rows: the edge lengths, and
    # sequences of up to 300 rows to the wanted total
    limit = 3072 if causal else 2048
    total = {0: limit, 1: limit + 1, 2400: limit + 2400}[extra]
    lengths = list(EDGES)
    while sum(lengths) < total:
        lengths.append(min(300, total - sum(lengths)))
    sizes, texts = _split_edges(lengths)
    X, img_off, E, text_off, params = _case(40 + causal, D, 128, sizes, texts)
    got = _run(D, 128, X, img_off, E, text_off, params, causal=causal)
    images = list(range(len(EDGES))) + [len(lengths) - 1]
    exact = _oracle(X, img_off, E, text_off, params, causal=causal, images=images)
    mirror = _oracle(X, img_off, E, text_off, params, causal=causal, mirror=True, images=images)
    rows = np.concatenate([np.arange(img_off[b], img_off[b + 1]) for b in images])
    _check(f"{total} rows {'causal' if causal else 'bidirectional'}", got[rows],
           np.concatenate([exact[b] for b in images]), np.concatenate([mirror[b] for b in images]))


@pytest.mark.parametrize("causal", [False, True], ids=["bidirectional", "causal"])
def test_shared_keys(gpu_lib, causal):
    """Sequences past the line, with two short ones among them."""
    first = 769 if causal else 513
    lengths = [first, first + 30, 33, first + 31, first + 62, first + 63, first + 64, 100, first + 127]
    sizes, texts = _split_edges(lengths)
    X, img_off, E, text_off, params = _case(42 + causal, 2048, 128, sizes, texts)
    got = _run(2048, 128, X, img_off, E, text_off, params, causal=causal)
    images = [0, 1, 2, 4, 5, 7, 8]
    exact = _oracle(X, img_off, E, text_off, params, causal=causal, images=images)
    print("exact done", flush=True)
    mirror = _oracle(X, img_off, E, text_off, params, causal=causal, mirror=True, images=images)
    rows = np.concatenate([np.arange(img_off[b], img_off[b + 1]) for b in images])
    _check(f"shared keys {'causal' if causal else 'bidirectional'}", got[rows],
           np.concatenate([exact[b] for b in images]), np.concatenate([mirror[b] for b in images]))
