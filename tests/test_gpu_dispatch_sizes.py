"""Dispatch at the sizes where its launches change: one block (with and without the row
copy), the folded scan, the separate scans; pair counts around a wave, a block round and the
limits, expert counts up to the largest; dead experts, and every pair on one expert.
Against a stable sort by expert: every output exact, rows past the last pair untouched."""
import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu

# T, k, d, M, D, p_alive, one_expert
CASES = [
    (1, 1, 1, 1, 64, 1.0, False), (1, 8, 2, 32, 64, 0.5, False), (8, 4, 2, 32, 1024, 1.0, False),
    (63, 1, 2, 4, 64, 0.9, False), (13, 5, 3, 5, 128, 0.9, True), (341, 3, 1, 128, 192, 0.8, False),
    (1023, 1, 2, 64, 64, 0.9, False), (205, 5, 2, 64, 64, 1.0, True), (512, 4, 3, 20, 256, 0.9, False),
    (2049, 1, 2, 4, 64, 0.9, False), (1025, 2, 1, 90, 64, 0.0, False), (4096, 4, 2, 32, 64, 0.9, False),
    (98305, 2, 1, 4, 64, 0.9, False), (98304, 2, 2, 3, 64, 0.9, False), (1250, 4, 2, 64, 64, 0.9, False),
    (700, 3, 2, 64, 64, 0.9, True), (4099, 8, 2, 31, 64, 0.95, False), (5000, 8, 2, 64, 64, 0.9, False),
    (200, 8, 3, 25, 64, 0.9, False), (33, 2, 3, 25, 64, 0.9, False), (100, 4, 2, 64, 64, 0.9, False),
]


@pytest.mark.parametrize("T,k,d,M,D,p_alive,one_expert", CASES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_dispatch(dtype, T, k, d, M, D, p_alive, one_expert):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(T * 7 + k)
    N, P, dev = M ** d, T * k, torch.device("cuda:0")
    idx = torch.randint(0, N, (T, k), generator=gen).to(torch.int32)
    alive = (torch.rand(N, generator=gen) < p_alive).to(torch.uint8)
    if one_expert:
        idx.fill_(N - 1)
        alive[N - 1] = 1
    x = torch.randn(T, D, generator=gen).to(dt)
    dims = abi.make_dims(T, D, 64, d, M, k, dtype, "relu")
    ws = torch.full((abi.ffn_workspace_bytes(dims) + 256,), 255, dtype=torch.uint8, device=dev)   # 256 past its end
    i32 = lambda *s: torch.full(s, -7, dtype=torch.int32, device=dev)
    counts, offsets, row_token, pos = i32(N), i32(N + 1), i32(P), i32(T, k)
    xp = torch.full((P, D), 9.0, dtype=dt, device=dev)
    abi.dmoe_dispatch(dims, x.to(dev), idx.to(dev), alive.to(dev), counts, offsets, row_token, pos, xp, ws)
    torch.cuda.synchronize()
    assert bool((ws[-256:] == 255).all())
    e = idx.view(-1).long()
    e = torch.where(alive[e] != 0, e, torch.full_like(e, N))
    order = torch.sort(e, stable=True)[1]
    rows = int((e < N).sum())
    rpos = torch.full((P,), -1, dtype=torch.int32)
    rpos[order[:rows]] = torch.arange(rows, dtype=torch.int32)
    cnt = torch.bincount(e, minlength=N + 1)[:N].to(torch.int32)
    assert torch.equal(counts.cpu(), cnt)
    assert torch.equal(offsets.cpu(), torch.cat([torch.zeros(1, dtype=torch.int32), cnt.cumsum(0).to(torch.int32)]))
    assert torch.equal(pos.cpu().view(-1), rpos)
    tok = (order[:rows] // k).to(torch.int32)
    assert torch.equal(row_token.cpu()[:rows], tok) and bool((row_token[rows:] == -7).all())
    assert torch.equal(xp.cpu()[:rows], x[tok.long()]) and bool((xp[rows:] == 9.0).all())
