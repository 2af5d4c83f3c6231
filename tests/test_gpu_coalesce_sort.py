"""Coalescing across the batch sizes where its sort, heads and sums change form
(GPU), against exact sums: whole-number signals whose sums every order gives."""
import numpy as np
import pytest
import torch

em = pytest.importorskip("paper_2607_01455_amd.ember")
DEV = "cuda"


def batch(P, V, kind, rng):
    if kind == "zipf":
        return np.minimum(rng.zipf(1.2, P) - 1, V - 1).astype(np.int64)
    if kind == "same":
        return np.full(P, V - 1, np.int64)
    if kind == "down":
        return (np.arange(P - 1, -1, -1, dtype=np.int64) % V).copy()
    return rng.integers(max(0, V - 3 * P), V, P).astype(np.int64)     # "high"


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["zipf", "same", "down", "high"])
@pytest.mark.parametrize("P", [1, 63, 64, 65, 1024, 1025, 2049, 4096, 4097, 6145, 16385, 40000, 65536, 65537])
def test_sort_and_heads(P, kind):
    V = 2 ** 31 - 2 if kind == "high" else 50021
    D = 5
    rng = np.random.default_rng(P)
    tok = batch(P, V, kind, rng)
    U = torch.from_numpy(rng.integers(-8, 9, (P, 8)).astype(np.float32)).to(DEV)[:, :D]
    co = em.Coalescer(P + 1000, V, D, dtype=torch.float32, device=DEV)   # workspace of a larger batch
    print(f"coalesce P={P} {kind}", flush=True)
    idx, G = co(torch.from_numpy(tok).to(DEV), U)
    want, inv = np.unique(tok, return_inverse=True)
    assert np.array_equal(idx.cpu().numpy(), want)
    sums = np.zeros((want.size, D))
    np.add.at(sums, inv, U.cpu().numpy().astype(np.float64))
    assert np.array_equal(G.cpu().numpy().astype(np.float64), sums)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [1, 2, 3, 255, 257, 1023, 1026])
@pytest.mark.parametrize("ud,gd", [(torch.float32, torch.float32), (torch.bfloat16, torch.bfloat16),
                                   (torch.bfloat16, torch.float32), (torch.float32, torch.bfloat16)])
def test_ragged_columns(D, ud, gd):
    P, V = 700, 300
    rng = np.random.default_rng(D)
    tok = rng.integers(0, V, P).astype(np.int64)
    q = 8
    ld = (D + q - 1) // q * q
    U = torch.full((P, ld), float("nan"), dtype=ud, device=DEV)          # padding must not matter
    U[:, :D] = torch.from_numpy(rng.integers(-4, 5, (P, D)).astype(np.float32)).to(DEV).to(ud)
    co = em.Coalescer(P, V, D, dtype=gd, device=DEV)
    pad = co.G_rows._base if co.G_rows._base is not None else co.G_rows
    pad.fill_(7.0)
    print(f"coalesce D={D}", flush=True)
    idx, G = co(torch.from_numpy(tok).to(DEV), U[:, :D])
    want, inv = np.unique(tok, return_inverse=True)
    sums = np.zeros((want.size, D))
    np.add.at(sums, inv, U[:, :D].float().cpu().numpy().astype(np.float64))
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(G.float().cpu().numpy().astype(np.float64), sums)   # |sum| <= 256: exact in bf16
    assert bool((pad[:, D:] == 7.0).all()), "columns past D were written"
    assert bool((pad[want.size:, :D] == 7.0).all()), "rows past n were written"


@pytest.mark.parametrize("D", [1, 64, 1023, 4096, 8192])
def test_workspace_covers_every_smaller_batch(D):
    sizes = sorted({max(1, int(x)) for x in np.geomspace(1, 1 << 20, 400)}
                   | {16 * k for k in (1, 511, 512, 513, 1024)} | {48 * 4096, 48 * 4096 + 1, 65536, 65537})
    got = [em.ember_coalesce_workspace_bytes(P, 50000, D) for P in sizes]
    assert all(a <= b for a, b in zip(got, got[1:]))
