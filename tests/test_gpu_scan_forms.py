"""The scan for any (K, L), its layouts for one, two, four and eight heads per KV head, and the lengths of
its runs: table sets whose last group is full, short or everything, key codes that end anywhere in a
16-byte group of words, against the oracle; and the step with the least scratch it is promised to run with."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import binding as mp
from paper_2410_16179_amd import workloads as wl
from tests.gpu_helpers import Session, rel_err
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,Hq,Hkv,n,tau,dtype,kv", [
    (9, 110, 3, 3, 1337, 2, "bf16", ""), (8, 90, 4, 2, 700, 2, "bf16", "fp8"), (10, 300, 8, 2, 900, 2, "bf16", ""),
    (10, 64, 5, 1, 640, 1, "bf16", ""), (11, 33, 8, 1, 515, 1, "fp32", ""), (7, 31, 6, 2, 450, 2, "bf16", ""),
    (13, 40, 2, 2, 300, 1, "bf16", ""), (6, 97, 2, 1, 333, 3, "fp32", ""), (2, 2, 1, 1, 200, 2, "bf16", ""), (9, 100, 7, 1, 129, 2, "bf16", "")])
def test_any_table_set(oracle, K, L, Hq, Hkv, n, tau, dtype, kv):
    w = wl.Workload("any", 1, Hq, Hkv, n, K, L, dtype, (8,), min_hits=tau, kv=kv)
    run_case(oracle, w, indexed=(64,))


@pytest.mark.parametrize("b,hq,hkv,n,K,L", [(3, 40, 8, 14000, 10, 220), (1, 32, 32, 20011, 9, 110), (4, 32, 8, 21000, 9, 100),
                                            (2, 16, 16, 9000, 10, 150), (1, 8, 8, 4100, 8, 90)])
def test_least_scratch_gives_the_same_step(b, hq, hkv, n, K, L):
    print(f"[case] least scratch B={b} Hq={hq} Hkv={hkv} n={n} K={K} L={L}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    mu = 2 * rnd(b, hkv, 128)
    Kc = (rnd(b, hkv, n, 128) + mu[:, :, None]).to(torch.bfloat16)
    Vc, q = rnd(b, hkv, n, 128).to(torch.bfloat16), rnd(b, hq, 128).to(torch.bfloat16)
    W = rnd(128, K * L).to(torch.bfloat16)
    p = mp.make_params(batch=b, n_q_heads=hq, n_kv_heads=hkv, K=K, L=L, n_ctx=n, dtype="bf16")
    kc, qc, ws = mp.alloc_key_codes(p), mp.alloc_query_codes(p), mp.alloc_workspace(p)
    mp.magicpig_hash_keys(p, Kc, mu, W, 0, n, kc, ws)
    mp.magicpig_hash_query(p, q, W, qc, ws)
    nblk, units = (n + 63) // 64, b * hkv
    wb = next((x for x in range(1, 6) if units * -(-nblk // (4 * x)) <= 780), 6)
    partials = max(-(-nblk // (4 * wb)), -(-nblk // 16) + 3, -(-nblk // 256) * 16)
    need = (b * hq * partials * 528 + 255) // 256 * 256
    outs = []
    for scratch in (ws, torch.empty(need, dtype=torch.uint8, device="cuda"), None):
        out = torch.full((b, hq, 128), float("nan"), device="cuda")
        if scratch is None:
            mp.magicpig_sampled_attention_noalloc(p, q, Kc, Vc, mu, kc, qc, out)
        else:
            mp.magicpig_sampled_attention(p, q, Kc, Vc, mu, kc, qc, out, workspace=scratch)
        outs.append(out.cpu().numpy())
    # the same sample, the same arithmetic, other partial sums (float32, a few hundred keys)
    assert rel_err(outs[1], outs[0]) <= 1e-5
    np.testing.assert_array_equal(outs[2], outs[0])
