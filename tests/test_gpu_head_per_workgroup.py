"""The one-launch scan + gather of short contexts, a workgroup for each query head, against its form with debug
outputs (a workgroup for the heads of a KV head) and the oracle: two to eight heads per KV head, compiled and other
table sets, contexts of a few keys, on either side of the limit in workgroups, and lengths in device memory with
strided caches."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import workloads as wl
from tests.gpu_helpers import TOL, Session, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,n,K,L,tau,dtype,kv", [
    (1, 4, 1, 70, 10, 150, 2, "bf16", ""), (2, 8, 4, 1001, 9, 120, 1, "bf16", "fp8"), (1, 32, 8, 2048, 10, 150, 2, "bf16", ""),
    (1, 24, 8, 1300, 8, 75, 2, "fp32", ""), (1, 16, 2, 4096, 10, 170, 2, "bf16", ""), (2, 10, 2, 777, 10, 220, 3, "bf16", ""),
    (1, 7, 1, 1500, 9, 110, 2, "bf16", ""), (2, 6, 2, 515, 11, 33, 1, "fp32", ""), (1, 40, 8, 1600, 10, 100, 2, "bf16", "fp8"),
    (1, 32, 8, 6144, 9, 120, 2, "bf16", ""), (1, 32, 8, 6209, 9, 120, 2, "bf16", ""), (1, 2, 1, 3, 10, 150, 2, "bf16", "")])
def test_head_per_workgroup(oracle, B, Hq, Hkv, n, K, L, tau, dtype, kv):
    print(f"[case] head per workgroup B={B} Hq={Hq} Hkv={Hkv} n={n} K={K} L={L} {dtype} {kv}", flush=True)
    w = wl.Workload("heads", B, Hq, Hkv, n, K, L, dtype, (8,), min_hits=tau, kv=kv)
    data = wl.generate(w)
    mu = data["K"].mean(2).astype(np.float32)
    s = Session(K=K, L=L, dtype=dtype, Kc=data["K"], Vc=data["V"], q=data["q"], W=data["W"], min_hits=tau, kv=kv)
    s.set_mu(mu)
    s.hash_keys()
    s.hash_query()
    both = s.attend()
    s.ws.fill_(255)                                          # (partials that nobody wrote are NaN)
    one = s.attend(debug=False)
    # the same keys and weights; float32 sums may be taken in another order
    assert rel_err(one["out"], both["out"]) <= 1e-5
    last = (B - 1, Hq - 1)
    ref = oracle.decode_step(data["q"], data["K"], data["V"], data["W"], K, L, mu=mu, min_hits=tau, heads=[(0, 0), last])
    for b, h in {(0, 0), last}:
        assert rel_err(one["out"][b, h][None], ref["out"][b, h][None]) <= TOL


@pytest.mark.parametrize("B,Hq,Hkv,n,K,L,dtype,kv", [
    (1, 32, 8, 2000, 10, 150, "bf16", ""), (2, 10, 2, 1500, 9, 110, "bf16", "fp8"), (1, 8, 1, 3000, 8, 75, "fp32", ""), (1, 6, 3, 900, 10, 100, "bf16", "")])
def test_length_in_device_memory_and_strided_caches(B, Hq, Hkv, n, K, L, dtype, kv):
    w = wl.Workload("heads", B, Hq, Hkv, n, K, L, dtype, (8,), min_hits=2, kv=kv)
    data = wl.generate(w)
    live = torch.tensor([n], dtype=torch.int64, device="cuda")
    same = dict(K=K, L=L, dtype=dtype, Kc=data["K"], Vc=data["V"], q=data["q"], W=data["W"], min_hits=2, kv=kv)
    strided = Session(**same, n_ctx_dev=live, layout="token_major")
    strided.set_mu(data["K"].mean(2).astype(np.float32))
    strided.hash_keys()
    strided.hash_query()
    for m in (n, n - 1, n // 2 + 7, 64, 5):
        print(f"[case] head per workgroup Hq={Hq} Hkv={Hkv} n={m} of {n} K={K} L={L} {dtype} {kv} strided", flush=True)
        live.fill_(m)
        strided.ws.fill_(255)
        got = strided.attend(debug=False)["out"]
        # the same length given by the host, dense caches, a workgroup for the heads of a KV head
        dense = Session(**same, n_ctx=m)
        dense.mu, dense.key_codes, dense.q_codes = strided.mu, strided.key_codes, strided.q_codes
        want = dense.attend()["out"]
        if m == n:                                           # the same runs: the same sums in the same order
            np.testing.assert_array_equal(got, want)
        else:
            assert rel_err(got, want) <= 1e-5
