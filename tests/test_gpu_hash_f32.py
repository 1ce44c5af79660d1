"""float32 key hashing on the matrix cores against the oracle, bit for bit: ragged ranges of keys around
the 32-key tile and the 64-key block, every kind of last table group, strided caches, and rows that sit
on a hyperplane (the exact re-evaluation decides them)."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import binding as mp
from tests.gpu_helpers import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,units,n,first,layout,use_mu", [
    (8, 75, 1, 200, 0, "dense", True), (10, 33, 2, 331, 37, "dense", True), (16, 40, 1, 160, 31, "token_major", True),
    (1, 1, 3, 130, 1, "dense", False), (3, 32, 1, 193, 64, "dense", True), (5, 70, 2, 257, 0, "token_major", False),
    (12, 64, 1, 129, 0, "dense", True)])
def test_float32_key_codes(oracle, K, L, units, n, first, layout, use_mu):
    print(f"[case] f32 codes K={K} L={L} units={units} n={n} first={first} {layout} mu={use_mu}", flush=True)
    rng = np.random.default_rng(K * L + n)
    W = rng.standard_normal((128, K * L)).astype(np.float32)
    mu = (2 * rng.standard_normal((1, units, 128))).astype(np.float32) if use_mu else None
    Kc = rng.standard_normal((1, units, n, 128)).astype(np.float32) + (mu[:, :, None] if use_mu else 0)
    Kc = Kc.astype(np.float32)
    Kc[0, 0, first + 3] = mu[0, 0] if use_mu else 0                      # every projection exactly zero
    Kc[0, 0, first + 5] = (mu[0, 0] if use_mu else 0) + np.float32(1e-6) * W[:, 0]
    Kc[0, 0, first + 7] = np.float32(3e20) * np.sign(W[:, K * L - 1])    # huge values
    Kc[0, -1, first + 8] = np.float32(2e-30) * W[:, K * L // 2]          # tiny ones
    s = Session(K=K, L=L, dtype="fp32", Kc=Kc, Vc=Kc, q=np.zeros((1, units, 128), np.float32), W=W, layout=layout)
    s.set_mu(mu)
    s.key_codes.fill_(0x13572468)
    s.hash_keys(first, n - first)
    for g in range(units):
        want = oracle.hash_keys(Kc[0, g, first:], W, mu[0, g] if use_mu else None, K, L)
        np.testing.assert_array_equal(s.key_table_codes_unit(0, g)[first:], want)
    # the words of other keys stay as they were
    raw = s.key_codes.cpu().numpy().view(np.uint32)
    idx = mp.key_code_gather_index(s.params)[0, :, :first]
    assert (raw[idx] == 0x13572468).all()
