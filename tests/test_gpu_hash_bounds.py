"""Hash bits where the error bounds that decide what is re-evaluated exactly are hardest pressed: every
form of the hashing against the oracle, bit for bit."""
import numpy as np
import pytest

from paper_2410_16179_amd import workloads as wl
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


def _check_queries(oracle, rows, W, K, L, dtype):
    want = oracle.hash_query(rows, W, K, L)
    none = np.zeros((1, len(rows) // 8, 1, 128), np.float32)
    s = Session(K=K, L=L, dtype=dtype, Kc=none, Vc=none, q=rows[None], W=W)
    s.hash_query()
    np.testing.assert_array_equal(s.query_table_codes()[0], want, err_msg="queries, plain projector")
    s.prepare()
    s.q_codes.fill_(0)
    s.hash_query_prepared()
    np.testing.assert_array_equal(s.query_table_codes()[0], want, err_msg="queries, prepared projector")


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


def _near_hyperplanes(rng, W, n, scale):
    """n float32 rows of about `scale` per element, each orthogonal to one column of W up to its own rounding."""
    x = rng.standard_normal((n, 128))
    w = W.astype(np.float64)[:, rng.integers(0, W.shape[1], n)].T
    x -= w * ((x * w).sum(1) / (w * w).sum(1))[:, None]
    return (scale * x).astype(np.float32)


@pytest.mark.parametrize("xs,ws", [(2e-23, 1.0), (1e-25, 1.0), (2e-23, 1e8), (1.0, 2e-23), (1e9, 1e-24), (2e-23, 2e-23), (1e-19, 1e-19)])
def test_float32_norms_below_the_normal_range(oracle, xs, ws):
    # the squares of such elements underflow in float32: a bound from norms alone would be nothing
    print(f"[case] tiny norms, float32, {xs} {ws}", flush=True)
    K, L = 8, 20
    rng = np.random.default_rng(5)
    W = (ws * rng.standard_normal((128, K * L))).astype(np.float32)
    rows = _near_hyperplanes(rng, W, 330, xs)
    rows[7] = 0
    _check_keys(oracle, rows, W, None, K, L, "fp32")
    # the same distances to a centering vector of that size
    mu = (4 * xs * rng.standard_normal(128)).astype(np.float32)
    _check_keys(oracle, rows + mu, W, mu, K, L, "fp32")
    _check_queries(oracle, rows[:40], W, K, L, "fp32")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("e,we", [(-75, 0), (-80, 30), (-60, -80), (0, -75), (-75, -75), (-10, 20)])
def test_tiny_terms_that_a_large_pair_hides(oracle, dtype, e, we):
    # two elements of 2^e that cancel, 120 of -2^(e-27) and one that is 60 times as large, so that the sum is
    # -60 * 2^(e-27), or +60 * 2^(e-27), whatever a float32 sum in some order makes of it
    print(f"[case] hidden terms {dtype} {e} {we}", flush=True)
    K, L = 4, 40
    W = np.full((128, K * L), 2.0 ** we, np.float32)
    W[:, 1::2] *= -1
    rng = np.random.default_rng(1)
    rows = np.zeros((256, 128), np.float32)
    for i in range(len(rows)):
        at = rng.permutation(128)
        sign = 1.0 if i & 1 else -1.0
        rows[i, at[:2]] = 2.0 ** e, -(2.0 ** e)
        rows[i, at[2:122]] = sign * 2.0 ** (e - 27)
        rows[i, at[122]] = -sign * 60 * 2.0 ** (e - 27)
    _check_keys(oracle, rows, W, None, K, L, dtype)
    _check_queries(oracle, rows[:72], W, K, L, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_rows_that_are_not_finite_leave_the_others_alone(oracle, dtype):
    # the exact sums of the rows beside them (every third row cancels to nothing or nearly so) are untouched
    print(f"[case] infinite rows {dtype}", flush=True)
    K, L = 4, 40
    rng = np.random.default_rng(3)
    W = np.where(rng.random((128, K * L)) < 0.5, -1.0, 1.0).astype(np.float32)
    W[1] = W[0]
    rows = np.zeros((256, 128), np.float32)
    rows[0::3, :3] = 2.0 ** 60, -(2.0 ** 60), 2.0 ** -60
    rows[1::3] = rng.integers(-8, 9, (len(rows[1::3]), 128))
    rows[2::3, 4] = np.inf
    rows[2::6, 4] = -np.inf
    ok = np.isfinite(rows).all(1)
    want = oracle.hash_keys(rows[ok], W, None, K, L)
    s = Session(K=K, L=L, dtype=dtype, Kc=rows[None, None], Vc=rows[None, None], q=np.zeros((1, 1, 128), np.float32), W=W)
    s.hash_keys()
    np.testing.assert_array_equal(s.key_table_codes()[0, 0][ok], want)
    s.prepare()
    for code in (s.hash_keys, s.hash_keys_prepared):
        s.key_codes.fill_(0x5a5a5a5a)
        for first in range(0, 256, 64):
            code(first, 64)
        np.testing.assert_array_equal(s.key_table_codes()[0, 0][ok], want)


@pytest.mark.parametrize("K,L,heads,group", [(2, 40, 5, 8), (4, 33, 16, 4), (8, 75, 32, 2), (10, 40, 8, 8), (1, 70, 3, 8),
                                             (8, 416, 128, 8), (4, 416, 128, 8), (2, 512, 128, 8)])
def test_many_flagged_projections_of_a_few_vectors(oracle, K, L, heads, group):
    # keys that are their centering vector or next to it, queries whose large terms cancel: a wavefront lists more
    # than the 256 entries it has room for at once; with 128 heads there are more workgroups than compute units
    print(f"[case] flagged K={K} L={L} heads={heads} group={group}", flush=True)
    rng = np.random.default_rng(K * L + heads)
    W = rng.integers(-3, 4, (128, K * L)).astype(np.float32)
    W[1] = W[0]
    mu = rng.integers(-200, 201, (heads, 128)).astype(np.float32)
    keys = mu.copy()
    keys[1::4, 5] += 1
    keys[2::4, 9] -= 1
    keys[3::4] += rng.integers(-2, 3, keys[3::4].shape)
    q = rng.integers(-2, 3, (heads * group, 128)).astype(np.float32)
    hot = q[:: 12 if heads == 128 else 5]
    hot[:] = 0
    hot[:, :3] = 2.0 ** 60, -(2.0 ** 60), 1
    Kc = wl.store(keys, "bf16")[None, :, None]
    s = Session(K=K, L=L, dtype="bf16", Kc=Kc, Vc=Kc, q=q[None], W=W)
    s.set_mu(mu[None])
    s.prepare()
    s.q_codes.fill_(0)
    s.key_codes.fill_(0x5a5a5a5a)
    s.hash_keys_prepared(0, 1, q_codes=s.q_codes)
    np.testing.assert_array_equal(s.query_table_codes()[0], oracle.hash_query(q, W, K, L))
    got = s.key_table_codes()[0, :, 0]
    for h in range(heads):
        np.testing.assert_array_equal(got[h], oracle.hash_keys(Kc[0, h], W, mu[h], K, L)[0])
