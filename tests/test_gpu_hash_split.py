"""bf16 key hashing with the projector sweep split over one to eight grid layers (the fewer workgroups,
the more layers), at table shapes whose last group is long, short or everything, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import binding as mp
from tests.gpu_helpers import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,n", [(10, 150, 256 * 60 - 5), (9, 120, 256 * 110 - 1), (11, 65, 256 * 154 + 1), (4, 500, 256 * 200),
                                   (2, 32, 256 * 90 - 70), (8, 75, 256 * 300 - 33), (10, 33, 256 * 385 - 64), (16, 40, 255)])
def test_codes_of_a_split_sweep(oracle, K, L, n):
    print(f"[case] split sweep K={K} L={L} n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K * L)
    mu = 2 * torch.randn(1, 1, 128, generator=g, device="cuda")
    Kc = (torch.randn(1, 1, n, 128, generator=g, device="cuda") + mu[:, :, None]).to(torch.bfloat16)
    W = torch.randn(128, K * L, generator=g, device="cuda").to(torch.bfloat16)
    Kh = Kc.float().cpu().numpy()
    s = Session(K=K, L=L, dtype="bf16", Kc=Kh, Vc=Kh[:, :, :1].repeat(n, 2), q=np.zeros((1, 1, 128), np.float32),
                W=W.float().cpu().numpy())
    s.mu = mu
    s.key_codes.fill_(-1)
    s.hash_keys()
    rng = np.random.default_rng(n)
    rows = np.unique(np.concatenate([rng.integers(0, n, 250), np.arange(min(n, 3)), n - 1 - np.arange(min(n, 70))]))
    want = oracle.hash_keys(Kh[0, 0, rows], W.float().cpu().numpy(), mu[0, 0].cpu().numpy(), K, L)
    np.testing.assert_array_equal(s.key_table_codes_unit(0, 0, rows), want)
    assert not mp.hash_keys_stats(s.params, s.ws)["overflowed"]
