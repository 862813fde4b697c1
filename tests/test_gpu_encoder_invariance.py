"""What an image's encoding must not depend on, to the bit: rows that its
queries do not see, and how large a max_seq the caller passes.  Helpers of
test_gpu_encoder.py."""
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
