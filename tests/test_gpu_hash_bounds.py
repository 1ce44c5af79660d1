"""Hash bits where the error bounds that decide what is re-evaluated exactly are hardest pressed: every
form of the hashing against the oracle, bit for bit."""
import numpy as np
import pytest

from tests.gpu_helpers import Session

pytestmark = pytest.mark.gpu


def _check_keys(oracle, rows, W, mu, K, L, dtype, kv=""):
    """rows [n, 128], n > 128, through the prefill form and, 64 at a time, through the forms of a decode step."""
    n = len(rows)
    want = oracle.hash_keys(rows, W, mu, K, L)
    Kc = rows[None, None]
    s = Session(K=K, L=L, dtype=dtype, Kc=Kc, Vc=Kc, q=np.zeros((1, 1, 128), np.float32), W=W, kv=kv)
    s.set_mu(None if mu is None else mu[None, None])
    s.hash_keys()
    np.testing.assert_array_equal(s.key_table_codes()[0, 0], want, err_msg="prefill")
    s.key_codes.fill_(0x5a5a5a5a)
    for first in range(0, n, 64):
        s.hash_keys(first, min(64, n - first))
    np.testing.assert_array_equal(s.key_table_codes()[0, 0], want, err_msg="few keys, plain projector")
    s.prepare()
    s.key_codes.fill_(0x5a5a5a5a)
    for first in range(0, n, 64):
        s.hash_keys_prepared(first, min(64, n - first))
    np.testing.assert_array_equal(s.key_table_codes()[0, 0], want, err_msg="few keys, prepared projector")
    return want


@pytest.mark.parametrize("K,L", [(2, 3), (10, 150)])
@pytest.mark.parametrize("dtype,kv,big,tiny", [("bf16", "", 2.0 ** 30, 2.0 ** -30), ("bf16", "fp8", 2.0 ** 50, 2.0 ** -8),
                                               ("fp32", "", 2.0 ** 30, 2.0 ** -30)])
def test_centering_vector_that_cancels(oracle, K, L, dtype, kv, big, tiny):
    # mu.W_j is big + tiny - big: a float64 sum of it has lost the tiny part, which decides the sign
    print(f"[case] cancelling centering vector {dtype} {kv} K={K} L={L}", flush=True)
    W = np.ones((128, K * L), np.float32)
    mu = np.zeros(128, np.float32)
    mu[:3] = big, tiny, -big
    rows = np.zeros((200, 128), np.float32)
    rows[0::4, 0] = tiny / 2
    rows[1::4, 5] = 2 * tiny
    rows[2::4, 7] = tiny
    rows[3::4, :2] = tiny / 2, tiny
    want = _check_keys(oracle, rows, W, mu, K, L, dtype, kv)
    assert (want[0] == 0).all() and (want[1] == (1 << K) - 1).all()
