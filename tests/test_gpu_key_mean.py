"""The key mean around the sizes where its kernels change: a chunk of 256 rows, 32 chunks, caches beyond L2."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import binding as mp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,kv", [("bf16", ""), ("bf16", "fp8"), ("fp32", "")])
@pytest.mark.parametrize("b,h,n", [(1, 1, 1), (2, 3, 15), (1, 2, 255), (1, 1, 256), (3, 1, 257), (1, 2, 8192), (2, 1, 8193), (1, 5, 20011)])
def test_key_mean_at_its_edges(b, h, n, dtype, kv):
    print(f"[case] key mean {b} {h} {n} {dtype} {kv}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    k = (3 + torch.randn(b, n, h, 128, generator=g, device="cuda")).to({"bf16": torch.bfloat16, "fp32": torch.float32}[dtype])
    k = (k.to(torch.float8_e4m3fn) if kv else k).permute(0, 2, 1, 3)         # token by token
    p = mp.make_params(batch=b, n_q_heads=h, n_kv_heads=h, K=2, L=2, n_ctx=n, dtype=dtype, kv_dtype=kv, k_strides=k.stride()[:3])
    out = torch.full((b, h, 128), float("nan"), device="cuda")
    mp.magicpig_key_mean(p, k, out, mp.alloc_workspace(p))
    want = k.to(torch.float32).double().mean(2).cpu().numpy()
    # a thread adds 16 rows in float32 (16 roundings of 2^-24 of at most 16 max|k|, over 16 rows), the rest is float64
    assert np.abs(out.cpu().numpy() - want).max() <= 17 * 2.0 ** -24 * float(k.to(torch.float32).abs().max())
