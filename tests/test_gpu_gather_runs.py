"""The separate gather of the table form, its wavefronts taking several pieces of sixteen key blocks: lists
that carry keys from piece to piece, full batches, a last run that ends early, no samples at all, against the scan
of the same codes."""
import pytest
import torch

from paper_2410_16179_amd import binding as mp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,hq,hkv,n,K,L,tau,dtype,kv,indexed,live", [
    (8, 64, 8, 10300, 10, 150, 2, "bf16", "", 10240, 0),     # two pieces a run, six runs, the last one short
    (8, 64, 8, 10300, 6, 40, 1, "bf16", "", 9984, 9990),     # half of the keys sampled; the length in device memory
    (8, 64, 8, 10300, 12, 2, 2, "bf16", "fp8", 10300, 0),    # next to nothing sampled
    (10, 40, 8, 17000, 8, 75, 2, "fp32", "", 16960, 0),      # batches of sixteen rows
    (16, 64, 8, 35000, 9, 120, 2, "bf16", "fp8", 34944, 300), # eight pieces a run, most runs empty
])
def test_runs_of_several_pieces(b, hq, hkv, n, K, L, tau, dtype, kv, indexed, live):
    _compare(b, hq, hkv, n, K, L, tau, dtype, kv, indexed, live)


# static sets with wavefronts of their own, and the forms without code for full batches
@pytest.mark.parametrize("b,hq,hkv,n,K,L,tau,dtype,kv,indexed,live,sink,local", [
    (8, 64, 8, 1000, 10, 150, 2, "bf16", "", 960, 0, 4, 900),         # of 64 keys
    (1, 32, 8, 9000, 10, 150, 3, "bf16", "", 8960, 8000, 31, 4100),   # the length in device memory
    (1, 32, 8, 9000, 10, 150, 3, "bf16", "fp8", 8960, 777, 16, 4096), # shorter than the static set
    (1, 32, 8, 2500, 7, 150, 3, "bf16", "", 2432, 0, 30, 200),        # of 32 keys; lists of several batches
    (1, 16, 8, 3333, 9, 75, 3, "fp32", "", 3328, 0, 333, 3000),       # every key static
    (65, 4, 4, 200, 10, 100, 2, "bf16", "fp8", 192, 0, 1, 64),        # 65 keys for one run
    (16, 64, 8, 9000, 10, 150, 2, "bf16", "", 8960, 0, 0, 3000),      # of 128 keys, three pieces a run
    (1, 32, 8, 16384, 6, 100, 3, "fp32", "", 16384, 16001, 4, 64),    # dealt over the runs, most keys sampled
])
def test_large_static_sets(b, hq, hkv, n, K, L, tau, dtype, kv, indexed, live, sink, local):
    _compare(b, hq, hkv, n, K, L, tau, dtype, kv, indexed, live, n_sink=sink, n_local=local)


def _compare(b, hq, hkv, n, K, L, tau, dtype, kv, indexed, live, **static):
    print(f"[case] gather runs B={b} Hq={hq} n={n} K={K} L={L} tau={tau} {dtype} {kv} live={live} {static}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    at = torch.float32 if dtype == "fp32" else torch.bfloat16
    store = torch.float8_e4m3fn if kv else at
    mu = 2 * rnd(b, hkv, 128)
    Kc = torch.empty(b, hkv, n, 128, dtype=store, device="cuda")
    Vc = torch.empty_like(Kc)
    for i in range(b):
        Kc[i] = (rnd(hkv, n, 128) + mu[i, :, None]).to(store)
        Vc[i] = rnd(hkv, n, 128).to(store)
    q, W = rnd(b, hq, 128).to(at), rnd(128, K * L).to(at)
    same = dict(batch=b, n_q_heads=hq, n_kv_heads=hkv, K=K, L=L, n_cap=n, dtype=dtype, min_hits=tau, kv_dtype=kv, **static)
    n_dev = torch.tensor([live], dtype=torch.int64, device="cuda") if live else None
    p = mp.make_params(n_ctx=n, n_ctx_dev=n_dev, **same) if live else mp.make_params(n_ctx=n, **same)
    kc, qc, ws = mp.alloc_key_codes(p), mp.alloc_query_codes(p), mp.alloc_workspace(p)
    mp.magicpig_hash_keys(p, Kc, mu, W, 0, n, kc, ws)
    mp.magicpig_hash_query(p, q, W, qc, ws)
    built = min(indexed, live // 64 * 64) if live else indexed
    pb = mp.make_params(n_ctx=built, **same)
    tables = mp.alloc_tables(p)
    mp.magicpig_build_tables(pb, kc, tables, mp.alloc_table_build_workspace(pb))
    ws.fill_(255)                                            # (partials that nobody wrote are NaN)
    scan, got = (torch.full((b, hq, 128), float("nan"), device="cuda") for _ in range(2))
    mp.magicpig_sampled_attention_tables(p, q, Kc, Vc, mu, tables, built, kc, qc, got, workspace=ws)
    mp.magicpig_sampled_attention(p, q, Kc, Vc, mu, kc, qc, scan, workspace=ws)
    # the same keys and weights, float32 sums in another order (up to 20000 terms, errors of 2^-24 each that
    # mostly cancel): the bound of the other comparisons of the two forms
    err = ((got - scan).abs().amax(-1) / scan.abs().amax(-1)).max().item()
    assert err <= 1e-5, err
