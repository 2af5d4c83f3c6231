"""LM-head gradient GEMM at the edges of its token steps (token counts around
one step (32), a round of the stage ring (128) and the change of tile order
(4096)), with small integers as data, so that every fp32 sum is exact in any
order and G is the exact sum rounded once, bit for bit; and G's special values."""
import pytest
import torch

from parity_checks import B2, DEV, EPS, LR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V,D,gd", [
    (T, 300, 264, gd) for T in (31, 32, 33, 64, 95, 97, 128, 129, 161)
    for gd in (torch.float32, torch.bfloat16)
] + [
    (4096, 2305, 520, torch.float32),   # last of the wide groups, 10 x 3 tiles: groups of 8 and 2
    (4097, 2305, 520, torch.bfloat16),  # first of the narrow groups
    (33, 16389, 4096, torch.float32),   # past 256 MB of fp32 G: streamed, the last row tile ragged
    (96, 2001, 3072, torch.float32),    # 8 x 12 tiles, the last row tile ragged: narrow groups
    (96, 2001, 3080, torch.float32),    # 13 column tiles, and
    (96, 2048, 520, torch.bfloat16),    # whole row tiles, and
    (96, 2051, 520, torch.bfloat16),    # 9 row tiles: wide groups
])
def test_token_steps_are_exact(T, V, D, gd):
    from paper_2607_01455_amd import ember
    print(f"lmhead steps T={T} V={V} D={D} {gd}", flush=True)
    gen = torch.Generator().manual_seed(T + V)
    dY = torch.randint(-3, 4, (T, V), generator=gen).float()
    H = torch.randint(-3, 4, (T, D), generator=gen).float()
    ldv = (V + 7) // 8 * 8
    dYd = torch.full((T, ldv), float("nan"), dtype=torch.bfloat16, device=DEV)[:, :V]
    dYd.copy_(dY.to(DEV))
    G = torch.zeros(V, D, dtype=gd, device=DEV)
    W = torch.zeros(V, D, dtype=torch.bfloat16, device=DEV)
    tab = ember.EmberTable(V, D, device=DEV, lr=LR, beta2=B2, eps=EPS)
    tab.step_lmhead(W, dYd, H.bfloat16().to(DEV), G)
    torch.cuda.synchronize()
    want = (dY.t() @ H).to(gd)   # |sum| < 2^24: exact in fp32
    assert torch.equal(G.cpu(), want)
    # first step from zero state: r and c are (1 - beta2) times the mean squares
    # of the stored G; sums of up to 2305 fp32 squares in any order stay within
    # 2305 u < 1.4e-4, sums by halves as here within ~20 u
    sq = want.double().square()
    b2 = float(torch.tensor(B2, dtype=torch.float32))
    for got, ref in ((tab.r, sq.mean(1)), (tab.c, sq.mean(0))):
        ref = (1.0 - b2) * ref
        assert ((got.cpu().double() - ref).abs() <= 1e-5 * ref).all()


@pytest.mark.parametrize("V,D", [(256, 256), (70, 40)])     # a whole tile, and the checked epilogue
@pytest.mark.parametrize("gd", [torch.float32, torch.bfloat16])
def test_special_values_of_g(gd, V, D):
    # column j of H is one-hot-like, so G_ij adds at most three exact products:
    # bf16 midpoints and their neighbours, overflow, infinities, NaN, subnormals
    from paper_2607_01455_amd import ember
    big = 2.0 ** 127
    sums = [(1.0, 2.0 ** -8, 0.0), (1.0, 2.0 ** -8, 2.0 ** -20), (1.0, 2.0 ** -8, -2.0 ** -20), (1.0, 2.0 ** -7, 2.0 ** -8),
            (-1.0, -2.0 ** -8, -2.0 ** -20), (big * (2 - 2.0 ** -7), 2.0 ** 119, 0.0), (big * (2 - 2.0 ** -7), 2.0 ** 118, 0.0),
            (big, big, 0.0), (-big, -big, 0.0), (float("inf"), 1.0, 0.0), (float("inf"), float("-inf"), 0.0),
            (float("nan"), 1.0, 0.0), (2.0 ** -126, 0.0, 0.0), (2.0 ** -133, 0.0, 0.0), (-2.0 ** -130, 2.0 ** -133, 0.0),
            (0.0, 0.0, 0.0)]
    T = 3
    dY = torch.zeros(T, V)
    dY[:, :len(sums)] = torch.tensor(sums).t()
    H = torch.ones(T, D)
    H[:, 1] = -1.0
    G = torch.full((V, D), 5.0, dtype=gd, device=DEV)
    W = torch.zeros(V, D, dtype=torch.bfloat16, device=DEV)
    tab = ember.EmberTable(V, D, device=DEV, lr=LR, beta2=B2, eps=EPS)
    print(f"lmhead specials {gd} {V}x{D}", flush=True)
    dYd = torch.zeros(T, (V + 7) // 8 * 8, dtype=torch.bfloat16, device=DEV)[:, :V]
    dYd.copy_(dY.to(DEV))
    tab.step_lmhead(W, dYd, H.bfloat16().to(DEV), G)
    want32 = torch.zeros(V, D)
    for t in range(T):
        want32 += dY[t].bfloat16().float()[:, None] * H[t][None, :]
    want = want32.to(gd)
    got = G.cpu()
    nan = torch.isnan(want)
    assert torch.equal(torch.isnan(got), nan)
    assert torch.equal(got[~nan], want[~nan])
