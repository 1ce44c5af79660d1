"""Float32 key hashing in workgroups of 64 keys (five bits per table or more, more than 256 workgroups of 32) and of 32: ragged ends, one to
sixteen bits per table, full and short last table groups, against the oracle bit for bit."""
import numpy as np
import pytest

from paper_2410_16179_amd import binding as mp
from tests.gpu_helpers import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("units,n,first,K,L", [
    (3, 1700, 0, 8, 75), (3, 1701, 33, 9, 65), (5, 1003, 95, 16, 64), (5, 1690, 64, 1, 33), (4, 901, 1, 11, 96),
    (2, 190, 31, 10, 150)])                                  # (one bit per table and the last one: workgroups of 32 keys)
def test_tiles(oracle, units, n, first, K, L):
    print(f"[case] f32 tiles units={units} n={n} first={first} K={K} L={L}", flush=True)
    rng = np.random.default_rng(K * L + n)
    W = rng.standard_normal((128, K * L)).astype(np.float32)
    mu = (2 * rng.standard_normal((1, units, 128))).astype(np.float32)
    Kc = (rng.standard_normal((1, units, n, 128)) + mu[:, :, None]).astype(np.float32)
    Kc[0, :, first + 2] = mu[0]                               # every projection is zero
    Kc[0, :, n - 1] = mu[0] + np.float32(1e-6) * W[:, 0]
    s = Session(K=K, L=L, dtype="fp32", Kc=Kc, Vc=Kc, q=np.zeros((1, units, 128), np.float32), W=W)
    s.set_mu(mu)
    s.key_codes.fill_(0x13572468)
    s.hash_keys(first, n - first)
    for g in (0, units - 1):
        np.testing.assert_array_equal(s.key_table_codes_unit(0, g)[first:], oracle.hash_keys(Kc[0, g, first:], W, mu[0, g], K, L))
    raw = s.key_codes.cpu().numpy().view(np.uint32)           # the words of other keys stay as they were
    assert (raw[mp.key_code_gather_index(s.params)[0, :, :first]] == 0x13572468).all()
