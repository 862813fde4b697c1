"""What an image's encoding must not depend on, to the bit: rows that its
queries do not see, how large a max_seq the caller passes, and what else is in
the batch.  Helpers of test_gpu_encoder.py."""
import numpy as np
import pytest

from tests.test_gpu_encoder import _case, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [700, 3100], ids=["keys_split", "keys_shared"])
def test_causal_rows_do_not_see_a_later_nan(gpu_lib, rows):
    """A NaN in a later 32-key block leaves a causal query's row as it is (a
    masked key in the query's own block is weighted with 0, which keeps a NaN)."""
    X, img_off, E, text_off, params = _case(61, 512, 128, (rows - 4,), (4,))
    want = _run(512, 128, X, img_off, E, text_off, params, causal=True)
    for p in (rows // 128 * 64 + 42, rows // 128 * 64 + 7):        # the later and the earlier half of 64 keys
        Y = X.copy()
        Y[p] = np.nan
        got = _run(512, 128, Y, img_off, E, text_off, params, causal=True)
        seen = p // 32 * 32
        np.testing.assert_array_equal(got[:seen], want[:seen])
        assert np.isnan(got[p:]).all()


@pytest.mark.parametrize("rows", [300, 2300], ids=["keys_split", "keys_shared"])
def test_any_max_seq_is_taken(gpu_lib, rows):
    """A max_seq far past the batch (no limit, to the caller) launches and gives the same bits."""
    X, img_off, E, text_off, params = _case(62, 512, 128, (rows - 4,), (4,))
    want = _run(512, 128, X, img_off, E, text_off, params)
    np.testing.assert_array_equal(_run(512, 128, X, img_off, E, text_off, params, max_seq=2**31 - 1), want)


@pytest.mark.parametrize("causal", [False, True], ids=["bidirectional", "causal"])
def test_an_image_encodes_alone_as_in_any_batch(gpu_lib, causal):
    """Images of few rows (keys split over the waves) and of many (keys shared),
    on both sides of the line (2048 rows at four heads, 3072 when causal): alone,
    in a batch of their own kind and mixed with the others."""
    edge = 3072 if causal else 2048
    totals = (300, 40, edge, edge + 1, 129, 1)
    texts = [min(9, n - 1) for n in totals]
    X, img_off, E, text_off, params = _case(63, 512, 128, [n - t for n, t in zip(totals, texts)], texts)

    def encode(images):
        x = np.concatenate([X[img_off[b]:img_off[b + 1]] for b in images])
        e = np.concatenate([E[text_off[b]:text_off[b + 1]] for b in images])
        io = np.cumsum([0] + [img_off[b + 1] - img_off[b] for b in images])
        to = np.cumsum([0] + [text_off[b + 1] - text_off[b] for b in images])
        H = _run(512, 128, x, io, e, to, params, causal=causal)
        return {b: H[io[i]:io[i + 1]] for i, b in enumerate(images)}

    mixed = encode(range(len(totals)))
    for group in [[0], [1], [2], [3], [0, 1, 4], [0, 3], [5, 2]]:
        for b, H in encode(group).items():
            np.testing.assert_array_equal(H, mixed[b], err_msg=f"image {b} of {group}")
