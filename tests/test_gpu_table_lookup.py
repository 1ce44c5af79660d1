"""The lookup for many heads (bitmaps of the whole indexed range): buckets of every length around what a
wavefront requests at once, few and many tables, against the scan of the same codes."""
import numpy as np
import pytest

from paper_2410_16179_amd import workloads as wl
from tests.gpu_helpers import Session, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,n,tau", [(10, 150, 700, 2), (6, 17, 2560, 2), (6, 40, 2600, 1), (5, 130, 3000, 2), (5, 8, 3100, 2),
                                       (4, 33, 3000, 2), (3, 5, 2000, 1), (8, 512, 700, 2), (9, 260, 2048, 2), (2, 3, 1500, 2)])
def test_lookup_of_many_heads(oracle, K, L, n, tau):
    print(f"[case] lookup K={K} L={L} n={n} tau={tau}", flush=True)
    w = wl.Workload("lookup", 9, 30, 5, n, K, L, "bf16", (8,), min_hits=tau)
    data = wl.generate(w)
    data["K"][:, :, : n // 3] = data["K"][:, :, :1]          # a third of the keys in one bucket of every table
    mu = data["K"].mean(2).astype(np.float32)
    s = Session(K=K, L=L, dtype="bf16", Kc=data["K"], Vc=data["V"], q=data["q"], W=data["W"], min_hits=tau)
    s.set_mu(mu)
    s.hash_keys()
    s.hash_query()
    scan = s.attend()
    for big in (True, False):                                # buckets ordered by window, and in no order
        s.build_tables(big_workspace=big)
        res = s.attend(tables=True, with_counts=False)
        np.testing.assert_array_equal(res["ncand"], scan["ncand"])
        for b in range(9):
            for h in range(30):
                np.testing.assert_array_equal(res["S"][b][h], scan["S"][b][h])
        assert rel_err(res["out"], scan["out"]) <= 1e-5
    ref = oracle.decode_step(data["q"], data["K"], data["V"], data["W"], K, L, mu=mu, min_hits=tau, heads=[(8, 29)])
    np.testing.assert_array_equal(scan["S"][8][29], ref["S"][8][29])
