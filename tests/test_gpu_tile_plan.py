"""The tile plan over many experts: experts with rows in the first, a middle and the last group of
64, on both sides of every 1024th, with row counts around the tile heights.  The plan steers every
tile of the expert GEMMs, so forward and backward of each expert with rows are compared with plain
products in fp64, and the gradients of the others have to stay untouched."""
import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,M,rows", [
    ("bf16", 2, 32, {0: 1, 63: 33, 64: 32, 511: 288, 1023: 289}),
    ("bf16", 3, 11, {0: 31, 127: 64, 1023: 5, 1024: 129, 1330: 40}),
    ("f32", 3, 11, {1: 65, 128: 1, 1023: 64, 1024: 63, 1330: 33}),
    ("bf16", 4, 11, {0: 3, 959: 32, 960: 1, 8191: 17, 14640: 33}),
    ("f32", 3, 25, {1023: 2, 1024: 40, 15624: 31}),
    ("bf16", 1, 3, {0: 600, 1: 1, 2: 700}), ("bf16", 2, 8, {q: 300 + 7 * q for q in range(64)}),
])
def test_experts_with_rows_are_found(dtype, d, M, rows):
    N, D, H, T = M ** d, 64, 128, sum(rows.values())
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(N + T)

    def rn(*s, scale=1.0):
        return (torch.randn(*s, generator=g, device="cuda") * scale).to(dt)

    counts = torch.zeros(N, dtype=torch.int32)
    for e, r in rows.items():
        counts[e] = r
    offsets = torch.cat([torch.zeros(1, dtype=torch.int32), counts.cumsum(0).int()]).cuda()
    counts = counts.cuda()
    dims = abi.make_dims(T, D, H, d, M, 1, dtype, "relu", 0)
    ws = torch.empty(abi.workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    x, dy = rn(T, D), rn(T, D)
    W1, b1, W2, b2 = rn(N, H, D, scale=D ** -0.5), rn(N, H), rn(N, D, H, scale=H ** -0.5), rn(N, D)
    h, a, dh = (torch.zeros(T, H, dtype=dt, device="cuda") for _ in range(3))
    y, dx = (torch.zeros(T, D, dtype=dt, device="cuda") for _ in range(2))
    grads = [torch.full_like(v, 7.0) for v in (W1, b1, W2, b2)]
    abi.dmoe_expert_ffn_fwd(dims, offsets, x, W1, b1, W2, b2, h, a, y, ws)
    abi.dmoe_expert_ffn_bwd(dims, offsets, counts, x, h, a, dy, W1, W2, dh, dx, *grads, ws)
    torch.cuda.synchronize()

    # one rounding of each stored tensor (bf16: 2^-9 relative), and of the fp32 sums
    tol = 2e-2 if dtype == "bf16" else 1e-5

    def close(got, ref):
        ref = ref.float()
        assert bool(((got.float() - ref).abs() <= tol * (ref.abs() + ref.square().mean().sqrt() + 1e-30)).all())

    for e in rows:
        s = slice(int(offsets[e]), int(offsets[e + 1]))
        close(h[s], x[s].double() @ W1[e].double().t() + b1[e].double())
        close(a[s], torch.relu(h[s]).double())
        close(y[s], a[s].double() @ W2[e].double().t() + b2[e].double())
        close(dh[s], (dy[s].double() @ W2[e].double()) * (h[s] > 0))
        close(dx[s], dh[s].double() @ W1[e].double())
        for got, ref in zip(grads, (dh[s].double().t() @ x[s].double(), dh[s].double().sum(0),
                                    dy[s].double().t() @ a[s].double(), dy[s].double().sum(0))):
            close(got[e], ref)
    rest = torch.ones(N, dtype=torch.bool, device="cuda")
    rest[list(rows)] = False
    assert all(bool((v[rest] == 7.0).all()) for v in grads)
