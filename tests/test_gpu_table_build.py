"""The window-ordered table build (count, offsets, place) against numpy at the sizes where it can go
wrong: every kind of tail string, table groups that start anywhere in a 16-byte group of words, tables
per workgroup that change with K, and contexts around a 64-key block and a 16384-key window."""
import numpy as np
import pytest
import torch

from paper_2410_16179_amd import binding as mp
from tests.gpu_helpers import pack_table_codes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,n,cap,units", [
    (10, 150, 16385, 16449, 2), (9, 120, 16384, 16384, 1), (10, 17, 63, 100, 3), (10, 8, 1, 1, 1), (8, 75, 20000, 20011, 2),
    (11, 41, 16447, 16500, 1), (12, 37, 33000, 33001, 1), (12, 3, 65, 200, 2), (9, 40, 0, 100, 1), (7, 33, 4097, 4097, 9), (5, 64, 1000, 1024, 1),
    (1, 512, 130, 130, 1), (3, 65, 129, 131, 2), (2, 31, 70, 70, 1), (6, 96, 16383, 16384, 1), (4, 40, 128, 128, 1)])
def test_window_ordered_build(K, L, n, cap, units):
    print(f"[case] build K={K} L={L} n={n} cap={cap} units={units}", flush=True)
    rng = np.random.default_rng(K * 1000 + L + n)
    codes = rng.integers(0, 1 << K, size=(units, cap, L))
    codes[:, : cap // 3, 1::2] = 5 % (1 << K)                # some buckets hold a third of the keys
    p = mp.make_params(batch=1, n_q_heads=units, n_kv_heads=units, K=K, L=L, n_ctx=n, n_cap=cap, dtype="bf16")
    raw = rng.integers(0, 1 << 32, size=mp.magicpig_key_code_bytes(p) // 4, dtype=np.uint32)   # (keys beyond cap: noise)
    raw[mp.key_code_gather_index(p)[0].ravel()] = mp.key_words_from_planes(pack_table_codes(codes, K, L, 0), K, L).ravel()
    tables = torch.full((mp.magicpig_table_bytes(p),), 0x5a, dtype=torch.uint8, device="cuda")
    mp.magicpig_build_tables(p, torch.from_numpy(raw.view(np.int32)).cuda(), tables, mp.alloc_table_build_workspace(p))
    got = tables.cpu().numpy().view(np.uint32)
    nb, windows = 1 << K, max(1, (n + 16383) // 16384)
    assert got[0] == windows
    at = 64
    off = got[at:at + units * L * (nb + 1)].reshape(units, L, nb + 1)
    at += (off.size * 4 + 255) // 256 * 64
    idx = got[at:at + units * L * cap].reshape(units, L, cap)
    at += (idx.size * 4 + 255) // 256 * 64
    fill = got[at:at + units * L * windows * nb].reshape(units, L, windows, nb)
    for u in range(units):
        for t in range(L):
            c = codes[u, :n, t]
            win = np.arange(n) >> 14
            counts = np.zeros((windows, nb), np.int64)
            np.add.at(counts, (win, c), 1)
            np.testing.assert_array_equal(off[u, t], np.concatenate([[0], np.cumsum(counts.sum(0))]))
            np.testing.assert_array_equal(fill[u, t], np.cumsum(counts, 0) - counts)
            # bucket by bucket, window by window; inside a piece in any order
            order = np.lexsort((np.arange(n), win, c))
            keys = idx[u, t, :n].astype(np.int64)
            np.testing.assert_array_equal(c[keys], c[order])
            np.testing.assert_array_equal(win[keys], win[order])
            np.testing.assert_array_equal(np.sort(keys), np.arange(n))
    assert (idx[:, :, n:] == 0x5a5a5a5a).all()               # nothing behind the keys
