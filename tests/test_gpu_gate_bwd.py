"""The gate's backward at the edges of its tiles: token counts around a stage (64 bf16 or 32
fp32 tokens), the 256-token groups, the dg blocks of 128 and the token splits; d_model with a
half column block; gate columns at the edges of the 32-column blocks; chosen experts that
share grid indices; dead experts; dg written over an input.  Against fp64: dg within fp32 rounding, dWg and dbg within
the stored type's rounding plus the error of fp32 sums of T terms (bf16: of terms carrying 16
mantissa bits) and of the terms themselves."""
import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu

CASES = [("bf16", T, D, d, M, k, pa) for T, D, d, M, k, pa in [
    (1, 64, 1, 2, 1, 1.0), (63, 128, 2, 4, 4, 0.8), (65, 192, 4, 3, 8, 0.9), (128, 64, 2, 16, 2, 1.0),
    (257, 320, 3, 11, 8, 0.9), (513, 64, 2, 48, 5, 0.7), (1100, 128, 2, 64, 8, 0.9), (2049, 64, 1, 128, 3, 1.0)]]
CASES += [("f32", T, D, d, M, k, pa) for T, D, d, M, k, pa in [
    (1, 64, 2, 2, 4, 1.0), (31, 192, 4, 4, 8, 0.8), (33, 64, 1, 33, 3, 1.0), (259, 128, 2, 40, 8, 0.9),
    (600, 64, 2, 64, 4, 0.9)]]
# splits of more than two 256-token groups: the terms of the third are loaded while the first is
# multiplied, and so on, up to a split's odd tail
DEEP = [("bf16", 20011, 2048, 2, 40, 8, 0.9), ("bf16", 8200, 4160, 4, 5, 3, 0.8), ("f32", 20011, 2048, 2, 20, 8, 0.9),
        ("f32", 16001, 2112, 3, 11, 5, 0.8)]


@pytest.mark.parametrize("dtype,T,D,d,M,k,p_alive", CASES + DEEP)
def test_gate_backward(dtype, T, D, d, M, k, p_alive):
    if T > 8000:                       # the split as the workspace lays it out
        split = max((T * ((D + 127) // 128) + 511) // 512, 256, 4 * d * M)
        assert (split + 63) // 64 * 64 > 512
    gen = torch.Generator().manual_seed(T + D + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    dev, dM, N = torch.device("cuda:0"), d * M, M ** d
    x = torch.randn(T, D, generator=gen).to(dt)
    # distinct experts, clustered so that grid indices repeat among a token's choices
    if T > 8000:
        idx = torch.rand(T, min(N, k + 6), generator=gen).argsort(1)[:, :k].to(torch.int32)
    else:
        idx = torch.stack([torch.randperm(min(N, k + 6), generator=gen)[:k] for _ in range(T)]).to(torch.int32)
    idx = (idx + torch.randint(0, max(1, N - k - 6), (T, 1), generator=gen)).to(torch.int32)
    w = torch.softmax(torch.randn(T, k, generator=gen), 1)
    dw = torch.randn(T, k, generator=gen)
    alive = (torch.rand(N, generator=gen) < p_alive).to(torch.uint8)
    dims = abi.make_dims(T, D, 64, d, M, k, dtype, "relu")
    # the workspace at its stated size, its contents poisoned
    ws = torch.full((abi.ffn_workspace_bytes(dims) + 256,), 255, dtype=torch.uint8, device=dev)   # 256 past its end
    dg = torch.empty(T, k, device=dev)
    dWg, dbg = torch.empty(dM, D, dtype=dt, device=dev), torch.empty(dM, dtype=dt, device=dev)
    abi.dmoe_gate_topk_bwd(dims, x.to(dev), idx.to(dev), w.to(dev), dw.to(dev), alive.to(dev), dg, dWg, dbg, ws)
    dWg2 = torch.empty_like(dWg)
    abi.dmoe_gate_topk_bwd(dims, x.to(dev), idx.to(dev), w.to(dev), dw.to(dev), alive.to(dev), dg, dWg2, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(dWg, dWg2)
    for which in (0, 1):                                 # dg written over w or over dw
        wd = [w.to(dev), dw.to(dev)]
        dWg3, dbg3 = torch.empty_like(dWg), torch.empty_like(dbg)
        abi.dmoe_gate_topk_bwd(dims, x.to(dev), idx.to(dev), wd[0], wd[1], alive.to(dev), wd[which], dWg3, dbg3, ws)
        torch.cuda.synchronize()
        assert bool((ws[-256:] == 255).all())
        assert torch.equal(wd[which], dg) and torch.equal(dWg, dWg3) and torch.equal(dbg, dbg3)
    wl = torch.where(alive[idx.long()] != 0, w, torch.zeros_like(w)).double()
    rdg = wl * (dw.double() - (wl * dw.double()).sum(1, keepdim=True))
    u = 2.0 ** -23
    # dg = w (dw - s), s = sum w dw in fp32: at most k roundings of s, one of the difference, one of
    # the product, so |error| <= (k + 2) u w (|dw| + sum w |dw|), also where dg cancels
    edg = (k + 2) * u * wl * (dw.double().abs() + (wl * dw.double().abs()).sum(1, keepdim=True))
    ds, eds = torch.zeros(T, dM, dtype=torch.float64), torch.zeros(T, dM, dtype=torch.float64)
    for i in range(d):
        ds.scatter_add_(1, idx.long() // M ** (d - 1 - i) % M + i * M, rdg)
        eds.scatter_add_(1, idx.long() // M ** (d - 1 - i) % M + i * M, edg)
    assert float((dg.cpu() - rdg).abs().max()) <= 4 * k * u * float((wl * dw.abs()).max() + 1)
    rel = 2.0 ** -8 if dtype == "bf16" else u            # rounding of the stored gradient
    for got, want, size, err in ((dWg, ds.t() @ x.double(), ds.abs().t() @ x.double().abs(), eds.t() @ x.double().abs()),
                                 (dbg, ds.sum(0), ds.abs().sum(0), eds.sum(0))):
        term = (T + 64) * u + (2.0 ** -16 if dtype == "bf16" and got is dWg else 0.0)
        lim = rel * want.abs() + (term + 8 * k * u) * (size + 1e-3) + err
        assert bool(((got.cpu().double() - want).abs() <= lim + 1e-7).all())
        # the limit leaves no room for a group of tokens lost or counted twice
        assert T < 2000 or float((got.cpu().double() - want).norm() / want.norm()) < (1e-2 if dtype == "bf16" else 1e-5)
