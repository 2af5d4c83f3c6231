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


# ---------------------------------------------------------------------------
# the order in which the rows of one id are added
# ---------------------------------------------------------------------------

BIG = 2.0 ** 60     # float64: 2^60 + 1 rounds back to 2^60


def ordered_batch(P, V, seed):
    """Ids of three positions each: a third of them side by side, a third within
    one run of 2048 positions, the rest anywhere in the batch.  Column j holds
    the 1 in the id's row j and +-2^60 in the other two, so a sum is 1 only if
    the row that was added last holds it: (0, 0, 1) in ascending order, and
    something else whenever another row comes last."""
    rng = np.random.default_rng(seed)
    slot = np.full(P, -1, np.int64)
    ids = 0

    def take(pool):
        nonlocal ids
        for k in range(0, pool.size - 2, 3):
            slot[pool[k:k + 3]] = ids
            ids += 1

    third = P // 3
    near = np.arange(0, third)
    take(near)
    mid = np.arange(third, 2 * third)
    for t in np.unique(mid // 2048):
        take(rng.permutation(mid[mid // 2048 == t]))
    take(rng.permutation(np.nonzero(slot < 0)[0]))
    alone = np.nonzero(slot < 0)[0]
    slot[alone] = ids + np.arange(alone.size)
    tok = rng.choice(V, ids + alone.size, replace=False).astype(np.int64)[slot]
    U = np.zeros((P, 4), np.float32)
    for p_of in np.split(np.argsort(slot, kind="stable")[:3 * ids], ids):
        p0, p1, p2 = np.sort(p_of)
        U[p0, :3], U[p1, :3], U[p2, :3] = (1, BIG, BIG), (BIG, 1, -BIG), (-BIG, -BIG, 1)
    U[:, 3] = rng.standard_normal(P)
    return tok, U, ids


def test_the_ordered_batch_tells_the_orders_apart():
    tok, U, ids = ordered_batch(1025, 50021, 1)
    triples = [np.nonzero(tok == t)[0] for t in np.unique(tok)]
    triples = [p for p in triples if p.size == 3]
    assert len(triples) == ids > 300

    def add(rows):
        s = np.zeros(3)
        for r in rows:
            s = s + U[r, :3].astype(np.float64)
        return s.tolist()

    for a, b, c in triples:
        assert add((a, b, c)) == [0.0, 0.0, 1.0]
        for other in ((a, c, b), (c, a, b), (b, c, a), (c, b, a)):   # every order with another row last
            assert add(other) != [0.0, 0.0, 1.0]


@pytest.mark.gpu
@pytest.mark.parametrize("V", [70001, 2 ** 21 + 5])
@pytest.mark.parametrize("P", [64, 1025, 2049, 4096, 4097, 16385, 65536, 65537])
@pytest.mark.parametrize("D", [3, 4])
def test_rows_of_an_id_are_added_in_position_order(P, D, V):
    import oracle
    tok, U, ids = ordered_batch(P, V, P)
    U = np.ascontiguousarray(U[:, :D])
    Ud = torch.zeros(P, 4, dtype=torch.float32, device=DEV)
    Ud[:, :D] = torch.from_numpy(U).to(DEV)
    co = em.Coalescer(P, V, D, dtype=torch.float32, device=DEV)
    print(f"coalesce order P={P} D={D} V={V}", flush=True)
    idx, G = co(torch.from_numpy(tok).to(DEV), Ud[:, :D])
    st, idx_o, G_o = oracle.coalesce(tok, U, V)
    assert st == oracle.OK and np.array_equal(idx.cpu().numpy(), idx_o)
    G = G.cpu().numpy()
    three = np.bincount(np.unique(tok, return_inverse=True)[1]) == 3
    assert three.sum() == ids
    assert np.array_equal(G[three, :3], np.tile(np.float32([0, 0, 1]), (ids, 1)))
    assert np.array_equal(G.view(np.uint32), G_o.view(np.uint32))
