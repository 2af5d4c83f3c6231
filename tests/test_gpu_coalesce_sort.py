"""Coalescing across the batch sizes where its sort, heads and sums change form
(GPU), against exact sums: whole-number signals whose sums every order gives."""
import ctypes

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


# ---------------------------------------------------------------------------
# which sort a batch of up to 64 sort tiles takes
# ---------------------------------------------------------------------------

SORT_TOKENS = (16384, 24576, 32768, 40960, 49152, 57344, 65536)
# radix minus counted sort, us, measured on an MI355X, by the table's id bits
RADIX_MINUS_COUNTED = {
    1: (-1.7, -4.6, -5.8, -14.4, -16.3, -21.2, -22.8),
    8: (0.0, -2.7, -4.8, -12.3, -15.1, -19.1, -21.4),
    9: (2.0, 0.6, -2.0, -8.0, -11.6, -13.0, -17.0),
    10: (5.7, 6.4, 3.0, -0.7, -5.2, -5.8, -9.0),
    11: (6.2, 3.9, 2.4, -4.3, -7.4, -10.7, -14.2),
    16: (8.8, 6.4, 4.8, -1.6, -4.7, -7.1, -11.0),
    17: (11.9, 12.8, 10.0, 6.5, 1.9, 3.4, -2.6),
    19: (18.2, 25.2, 20.1, 21.3, 14.7, 19.8, 13.4),
    21: (13.8, 14.5, 12.5, 5.5, 2.1, 1.3, -2.0),
    24: (18.2, 15.8, 14.5, 8.3, 5.6, 4.5, 1.0),
    31: (26.2, 25.4, 23.7, 17.8, 14.3, 15.6, 11.9),
}


def counted(P, V):
    fn = em.LIB._ZN5ember12coal_countedEll     # ember::coal_counted(int64_t, int64_t)
    fn.argtypes, fn.restype = [ctypes.c_int64, ctypes.c_int64], ctypes.c_bool
    return fn(P, V)


def test_each_batch_takes_the_faster_sort():
    for bits, row in RADIX_MINUS_COUNTED.items():
        V = min(2 ** bits, 2 ** 31 - 2)
        for P, d in zip(SORT_TOKENS, row):
            assert counted(P, V) == (d > 0) or abs(d) <= 2.0, (bits, P, d)
        for P in (1, 1000, 4096, 4097, 12288):
            assert counted(P, V)
        assert not counted(65537, V)


@pytest.mark.gpu
@pytest.mark.parametrize("P", [16385, 20000, 32768, 32769, 49152, 49153, 61441, 65536])
@pytest.mark.parametrize("V", [1, 2, 200, 257, 1000, 1500, 50021, 128256, 2 ** 20, 2 ** 21, 2 ** 21 + 1, 2 ** 31 - 2])
def test_both_sorts_of_up_to_64_tiles(P, V):
    D = 4
    rng = np.random.default_rng(P + V)
    tok = rng.integers(0, V, P).astype(np.int64)
    tok[rng.random(P) < 0.2] = V - 1                 # one frequent id
    U = torch.from_numpy(rng.integers(-8, 9, (P, D)).astype(np.float32)).to(DEV)
    co = em.Coalescer(P, V, D, dtype=torch.float32, device=DEV)
    print(f"coalesce P={P} V={V} counted={counted(P, V)}", flush=True)
    for bad_at in (P - 1, P // 2, 0):                # reported, and the workspace works on
        bad = tok.copy()
        bad[bad_at] = V if bad_at else -1
        em.ember_coalesce_rows(torch.from_numpy(bad).to(DEV), U, V, co.idx, co.G_rows, co.n_out, co.ws)
        assert em.ember_get_error(co.ws) == em.EMBER_ERR_INDEX and int(co.n_out.item()) == -1
    idx, G = co(torch.from_numpy(tok).to(DEV), U)
    want, inv = np.unique(tok, return_inverse=True)
    assert np.array_equal(idx.cpu().numpy(), want)
    sums = np.zeros((want.size, D))
    np.add.at(sums, inv, U.cpu().numpy().astype(np.float64))
    assert np.array_equal(G.cpu().numpy().astype(np.float64), sums)


@pytest.mark.gpu
@pytest.mark.parametrize("P", [65537, 70001])
@pytest.mark.parametrize("V", [1000, 2 ** 20, 2 ** 21 + 5, 2 ** 30, 2 ** 31 - 2])    # 1, 2, 3, 3 and 4 radix passes
def test_radix_passes_past_64_tiles(P, V):
    tok, U = np.random.default_rng(V).integers(0, V, P), np.random.default_rng(P).standard_normal((P, 4))
    tok[::7] = tok[3]
    U = torch.from_numpy(U.astype(np.float32)).to(DEV)
    co = em.Coalescer(P, V, 4, dtype=torch.float32, device=DEV)
    print(f"coalesce P={P} V={V}", flush=True)
    idx, G = co(torch.from_numpy(tok).to(DEV), U)
    want, inv = np.unique(tok, return_inverse=True)
    assert np.array_equal(idx.cpu().numpy(), want)
    U64 = U.cpu().numpy().astype(np.float64)
    sums, mags = np.zeros((want.size, 4)), np.zeros((want.size, 4))
    np.add.at(sums, inv, U64)
    np.add.at(mags, inv, np.abs(U64))
    # one rounding to fp32 of a float64 sum within (count - 1) 2^-53 sum|u| of the exact one, on both sides
    bound = 2.0 ** -24 * np.abs(sums) + 2 * P * 2.0 ** -53 * mags + 2.0 ** -149
    assert (np.abs(G.cpu().numpy().astype(np.float64) - sums) <= bound).all()


# ---------------------------------------------------------------------------
# special values through every form of the sums
# ---------------------------------------------------------------------------

@pytest.mark.gpu
@pytest.mark.parametrize("V", [40, 100003])     # fewer rows than positions, and more
@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 7, 255, 256, 257, 1021])
@pytest.mark.parametrize("ud,gd", [(torch.float32, torch.float32), (torch.bfloat16, torch.bfloat16),
                                   (torch.bfloat16, torch.float32), (torch.float32, torch.bfloat16)])
def test_special_values_in_every_form_of_the_sums(ud, gd, D, V):
    import oracle
    from parity_checks import bf16_values, host_bits
    from test_oracle_coalesce_pins import BF16_EDGE_SEGMENTS
    # fp32 bits of each id's rows; +-inf, NaN and -0 also in segments that chunks cut
    segs = [[b << 16 for b in rows] for rows, _ in BF16_EDGE_SEGMENTS]
    segs += [[0x7FC10000], [0x80000000] * 150, [0x3F800000] * 99 + [0x7F800000] + [0x3F800000] * 60,
             [0x7F800000] + [0x3F800000] * 120 + [0xFF800000], [0x00010000] * 130]
    if ud == torch.float32:
        segs += [[0x3F808008], [0x3F808000], [0x3F818000], [0x00000001], [0x00008001], [0x80000000],
                 [0x7F7FFFFF, 0x7F7FFFFF], [0x00000001] * 140]
    ids = np.sort(np.random.default_rng(D).choice(V, len(segs), replace=False)).astype(np.int64)
    tok = np.concatenate([np.full(len(r), k, np.int64) for k, r in zip(ids, segs)])
    rows = np.concatenate([np.array(r, np.uint64) for r in segs]).astype(np.uint32)
    perm = np.random.default_rng(9).permutation(tok.size)
    tok, rows = tok[perm], rows[perm]
    cols = np.stack([rows ^ (0x80000000 if j % 2 else 0) for j in range(D)], axis=1).astype(np.uint32)
    host = (cols >> 16).astype(np.uint16) if ud == torch.bfloat16 else cols.view(np.float32)
    q = 16 // torch.empty(0, dtype=ud).element_size()
    U = torch.full((tok.size, (D + q - 1) // q * q), float("nan"), dtype=ud, device=DEV)[:, :D]
    src = torch.from_numpy(host.view(np.int16) if ud == torch.bfloat16 else host).to(DEV)
    U.copy_(src.view(torch.bfloat16) if ud == torch.bfloat16 else src)
    co = em.Coalescer(tok.size, V, D, dtype=gd, device=DEV)
    pad = co.G_rows._base if co.G_rows._base is not None else co.G_rows
    pad.fill_(7.0)
    print(f"coalesce specials D={D} V={V} {ud}->{gd}", flush=True)
    idx, G = co(torch.from_numpy(tok).to(DEV), U)
    st, idx_o, want = oracle.coalesce(tok, host, V, out_dtype=np.uint16 if gd == torch.bfloat16 else np.float32)
    assert st == oracle.OK and np.array_equal(idx.cpu().numpy(), idx_o)
    got = host_bits(G)
    gv, wv = (bf16_values(got), bf16_values(want)) if gd == torch.bfloat16 else (got, want)
    nan = np.isnan(wv)
    assert np.array_equal(np.isnan(gv), nan)
    gb, wb = (got, want) if gd == torch.bfloat16 else (got.view(np.uint32), want.view(np.uint32))
    bad = np.argwhere((gb != wb) & ~nan)      # every sum is exact in float64: the same bits
    assert bad.size == 0, bad[:4].tolist()
    assert bool((pad[:, D:] == 7.0).all()) and bool((pad[ids.size:] == 7.0).all())


@pytest.mark.gpu
@pytest.mark.parametrize("D", [1, 2, 3, 5, 6, 7, 253, 254, 255, 257, 258, 259, 1027])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_last_row_may_end_with_the_storage(dt, D):
    # only the D columns of a row belong to it: U's storage ends with its last
    # element, and what the padding of the other rows holds does not matter
    P, V = 333, 100
    rng = np.random.default_rng(D)
    q = 16 // torch.empty(0, dtype=dt).element_size()
    ld = (D + q - 1) // q * q + q
    flat = torch.full(((P - 1) * ld + D,), float("nan"), dtype=dt, device=DEV)
    U = flat.as_strided((P, D), (ld, 1))
    U.copy_(torch.from_numpy(rng.integers(-4, 5, (P, D)).astype(np.float32)).to(DEV))
    tok = rng.integers(0, V, P).astype(np.int64)
    tok[-1] = V                                          # a segment of the last row alone
    co = em.Coalescer(P, V + 1, D, dtype=dt, device=DEV)
    print(f"coalesce tight D={D} {dt}", flush=True)
    idx, G = co(torch.from_numpy(tok).to(DEV), U)
    want, inv = np.unique(tok, return_inverse=True)
    sums = np.zeros((want.size, D))
    np.add.at(sums, inv, U.float().cpu().numpy().astype(np.float64))
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(G.float().cpu().numpy().astype(np.float64), sums)   # |sum| <= 256: exact in bf16
