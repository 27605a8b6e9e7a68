"""The column sums of the bias gradients at the edges of their row slices (16, 4 or 1 slices by
the average rows per expert, four rows of a slice in flight) and column blocks (16, 64 or 256
lanes of 8 bf16 or 4 fp32 columns): small integers, so every order of the fp32 sum is exact
and the result is known to the bit."""
import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu

COUNTS = {
    "many": [1, 0, 15, 16, 17, 48, 49, 63, 64, 65, 79, 80, 81, 129, 0, 200],
    "some": [1, 0, 3, 4, 5, 12, 13, 15, 16, 17, 31, 64, 32, 2, 0, 33],
    "few": [1, 0, 0, 3, 2, 1, 0, 17, 4, 1, 1, 0, 5, 0, 0, 2],
    "less_than_one": [0, 0, 0, 3, 0, 0, 0, 0, 1, 0, 0, 0, 0, 0, 0, 5],
}


@pytest.mark.parametrize("dtype,D,H", [("bf16", 64, 192), ("bf16", 192, 128), ("bf16", 64, 2112), ("bf16", 1088, 512),
                                       ("f32", 64, 128), ("f32", 128, 64), ("f32", 64, 1088)])
@pytest.mark.parametrize("rows", list(COUNTS))
def test_bias_gradients_are_exact_column_sums(rows, dtype, D, H):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    counts = COUNTS[rows]
    N, k, P = len(counts), 1, sum(counts)
    g = torch.Generator().manual_seed(5)
    dev = torch.device("cuda:0")
    dims = abi.make_dims(P, D, H, 2, 4, k, dtype, "relu")
    offs = torch.tensor([0] + counts, dtype=torch.int32).cumsum(0).to(torch.int32)
    dy = torch.randint(-2, 3, (P, D), generator=g).to(dt)
    e = lambda *s: torch.zeros(s, dtype=dt, device=dev)
    # W2 selects columns of dy (column h of dh is dy's column h % D) and h > 0 everywhere
    W2 = torch.zeros(N, D, H, dtype=dt)
    W2[:, torch.arange(H) % D, torch.arange(H)] = 1
    db1, db2 = torch.full((N, H), 7.0, dtype=dt, device=dev), torch.full((N, D), 7.0, dtype=dt, device=dev)
    ws = torch.empty(abi.workspace_bytes(dims), dtype=torch.uint8, device=dev)
    abi.dmoe_expert_ffn_bwd(dims, offs.to(dev), torch.tensor(counts, dtype=torch.int32, device=dev), e(P, D),
                            torch.ones(P, H, dtype=dt, device=dev), e(P, H), dy.to(dev), e(N, H, D), W2.to(dev),
                            e(P, H), e(P, D), e(N, H, D), db1, e(N, D, H), db2, ws)
    torch.cuda.synchronize()
    for x, c in enumerate(counts):
        want = dy[offs[x]:offs[x + 1]].double().sum(0).to(dt) if c else torch.full((D,), 7.0, dtype=dt)
        assert torch.equal(db2[x].cpu(), want), (dtype, x, c)
        want = want[torch.arange(H) % D] if c else torch.full((H,), 7.0, dtype=dt)
        assert torch.equal(db1[x].cpu(), want), (dtype, x, c)


@pytest.mark.parametrize("dtype,F", [("bf16", 64), ("bf16", 192), ("bf16", 2112), ("f32", 64), ("f32", 1088)])
@pytest.mark.parametrize("rows", list(COUNTS))
def test_layer_norm_parameter_gradients_are_exact(rows, dtype, F):
    """The same sums in the LayerNorm step's backward: with mean 0, deviation 1, scale 1 and
    shift 0 handed in, dgamma and dbeta are the column sums of da [h > 0] h and da [h > 0]."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    counts = COUNTS[rows]
    N, P, dev = len(counts), sum(counts), torch.device("cuda:0")
    g = torch.Generator().manual_seed(7)
    dims = abi.make_dims(P, 64, F, 2, 4, 1, dtype, "relu")
    offs = torch.tensor([0] + counts, dtype=torch.int32).cumsum(0).to(torch.int32)
    h, da = (torch.randint(-2, 3, (P, F), generator=g).to(dt) for _ in range(2))
    stats = torch.tensor([0.0, 1.0]).repeat(P, 1)
    dg, db = torch.full((N, F), 7.0, dtype=dt, device=dev), torch.full((N, F), 7.0, dtype=dt, device=dev)
    abi.dmoe_ln_act_bwd(dims, offs.to(dev), h.to(dev), stats.to(dev), torch.ones(N, F, dtype=dt, device=dev),
                        torch.zeros(N, F, dtype=dt, device=dev), da.to(dev), torch.empty(P, F, dtype=dt, device=dev), dg, db)
    torch.cuda.synchronize()
    dz = torch.where(h > 0, da, torch.zeros_like(da)).double()
    for x, c in enumerate(counts):
        s = slice(int(offs[x]), int(offs[x + 1]))
        for got, want in ((dg, (dz[s] * h[s].double()).sum(0)), (db, dz[s].sum(0))):
            assert torch.equal(got[x].cpu(), want.to(dt) if c else torch.full((F,), 7.0, dtype=dt)), (dtype, x, c)
