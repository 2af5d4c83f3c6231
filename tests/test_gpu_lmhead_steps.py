"""LM-head gradient GEMM at the edges of its token steps: token counts around
one step (32), a round of the stage ring (128) and the change of tile order
(4096), with small integers as data, so that every fp32 sum is exact in any
order and G is the exact sum rounded once, bit for bit."""
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
