"""The scan for any (K, L), its layouts for one, two, four and eight heads per KV head, and the lengths of
its runs: table sets whose last group is full, short or everything, key codes that end anywhere in a
16-byte group of words, against the oracle; and the step, bit for bit, with the least scratch it is promised
to run with."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import binding as mp
from paper_2410_16179_amd import workloads as wl
from tests.gpu_helpers import TOL, Session, rel_err
from tests.test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,Hq,Hkv,n,tau,dtype,kv", [
    (9, 110, 3, 3, 1337, 2, "bf16", ""), (8, 90, 4, 2, 700, 2, "bf16", "fp8"), (10, 300, 8, 2, 900, 2, "bf16", ""),
    (10, 64, 5, 1, 640, 1, "bf16", ""), (11, 33, 8, 1, 515, 1, "fp32", ""), (7, 31, 6, 2, 450, 2, "bf16", ""),
    (13, 40, 2, 2, 300, 1, "bf16", ""), (6, 97, 2, 1, 333, 3, "fp32", ""), (2, 2, 1, 1, 200, 2, "bf16", ""), (9, 100, 7, 1, 129, 2, "bf16", "")])
def test_any_table_set(oracle, K, L, Hq, Hkv, n, tau, dtype, kv):
    w = wl.Workload("any", 1, Hq, Hkv, n, K, L, dtype, (8,), min_hits=tau, kv=kv)
    run_case(oracle, w, indexed=(64,))


def _blocks_per_wavefront(b, hq, hkv, n):
    """Least scratch in partials per head, and key blocks per wavefront: those of the shortest runs that fit a round,
    and those of the runs taken."""
    nblk, units = -(-n // 64), b * hkv
    runs = lambda w: -(-nblk // (4 * w))                     # noqa: E731
    short = next((w for w in range(1, 6) if units * runs(w) <= 780), 6)
    most = max(runs(short), -(-nblk // 16) + 3, -(-nblk // 256) * 16)
    fit = [w for w in range(1, 7) if runs(w) <= most]
    at_once = [w for w in fit if units * runs(w) <= (1024 if hq == hkv else 780)] or [w for w in fit if units * runs(w) <= 1024]
    if at_once:
        return most, short, at_once[0]
    return most, short, min(fit, key=lambda w: (-(-units * runs(w) // 256) * (4 * w + 2), -w))


@pytest.mark.parametrize("b,hq,hkv,n,K,L,short,taken", [
    (1, 32, 32, 20011, 9, 110, 4, 3),                        # one head per KV head: shorter runs, two wavefronts share one
    (1, 8, 8, 28000, 9, 110, 2, 2), (1, 8, 8, 4100, 8, 90, 1, 1),
    (2, 16, 16, 9000, 10, 150, 2, 2),
    (8, 32, 8, 20000, 9, 100, 6, 5),                         # four workgroups per compute unit
    (3, 32, 8, 65536, 10, 120, 6, 4), (16, 64, 8, 16000, 9, 120, 6, 4)])   # several rounds
def test_the_step_does_not_depend_on_the_scratch(oracle, b, hq, hkv, n, K, L, short, taken):
    print(f"[case] least scratch B={b} Hq={hq} Hkv={hkv} n={n} K={K} L={L}", flush=True)
    partials, *form = _blocks_per_wavefront(b, hq, hkv, n)
    assert form == [short, taken]
    g = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    mu = 2 * rnd(b, hkv, 128)
    Kc = torch.empty(b, hkv, n, 128, dtype=torch.bfloat16, device="cuda")
    Vc = torch.empty_like(Kc)
    for i in range(b):
        Kc[i] = rnd(hkv, n, 128) + mu[i, :, None]
        Vc[i] = rnd(hkv, n, 128)
    q, W = rnd(b, hq, 128).to(torch.bfloat16), rnd(128, K * L).to(torch.bfloat16)
    p = mp.make_params(batch=b, n_q_heads=hq, n_kv_heads=hkv, K=K, L=L, n_ctx=n, dtype="bf16")
    kc, qc, ws = mp.alloc_key_codes(p), mp.alloc_query_codes(p), mp.alloc_workspace(p)
    mp.magicpig_hash_keys(p, Kc, mu, W, 0, n, kc, ws)
    mp.magicpig_hash_query(p, q, W, qc, ws)
    need = (b * hq * partials * 528 + 255) // 256 * 256
    outs = []
    for scratch in (ws, torch.empty(need, dtype=torch.uint8, device="cuda"), None):
        out = torch.full((b, hq, 128), float("nan"), device="cuda")
        if scratch is not None:
            mp.magicpig_sampled_attention(p, q, Kc, Vc, mu, kc, qc, out, workspace=scratch)
        elif need <= 8 << 20:
            mp.magicpig_sampled_attention_noalloc(p, q, Kc, Vc, mu, kc, qc, out)
        else:
            continue
        outs.append(out.cpu().numpy())
    for other in outs[1:]:
        np.testing.assert_array_equal(other, outs[0])
    G = hq // hkv
    for i, h in {(0, 0), (b - 1, hq - 1)}:                   # a first and a last head against the oracle
        u = (i, h // G)
        Kh, Vh = Kc[u].float().cpu().numpy(), Vc[u].float().cpu().numpy()
        ref = oracle.decode_step(q[i, h].float().cpu().numpy()[None, None], Kh[None, None], Vh[None, None], W.float().cpu().numpy(),
                                 K, L, mu=mu[u].cpu().numpy()[None, None])
        assert rel_err(outs[0][i, h][None], ref["out"][0]) <= TOL


@pytest.mark.parametrize("G,K,L,n", [(1, 9, 110, 2240), (2, 10, 300, 2177), (3, 8, 90, 2240), (5, 9, 100, 2200), (8, 11, 33, 2240)])
def test_appended_keys_scanned_on_their_own(oracle, G, K, L, n):
    # 33 or more key blocks behind the tables of 32 (batch, KV head) units: the scan alone, each layout of it
    print(f"[case] appended scan G={G} K={K} L={L} n={n}", flush=True)
    w = wl.Workload("appended", 8, 4 * G, 4, n, K, L, "bf16", (8,))
    data = wl.generate(w)
    s = Session(K=K, L=L, dtype="bf16", Kc=data["K"], Vc=data["V"], q=data["q"], W=data["W"])
    s.set_mu(data["K"].mean(2))
    s.hash_keys()
    s.hash_query()
    scan = s.attend()
    s.build_tables(64)
    res = s.attend(tables=True, with_counts=False)
    np.testing.assert_array_equal(res["ncand"], scan["ncand"])
    for b in range(8):
        for h in range(4 * G):
            np.testing.assert_array_equal(res["S"][b][h], scan["S"][b][h])
    assert rel_err(res["out"], scan["out"]) <= 1e-5
    ref = oracle.decode_step(data["q"], data["K"], data["V"], data["W"], K, L, mu=data["K"].mean(2), heads=[(7, 4 * G - 1)])
    np.testing.assert_array_equal(res["S"][7][4 * G - 1], ref["S"][7][4 * G - 1])
