"""The row-grouped bf16 GEMMs in each tile shape they can be given (by the average rows per
expert, the output width and the weights touched): experts without rows, with one row, with
counts either side of the 32-, 64-, 128- and 288-row tiles, widths that are no multiple of a
tile, and a heavy expert among light ones.  Forward, data gradients and weight gradients
against fp64 products on the GPU, elementwise |err| <= 2e-2 (|ref| + rms), the bf16 tolerance;
each stage from the library's own stored inputs to it."""
import ctypes

import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu

E = lambda *c: list(c)
CASES = {
    # few rows and few weights: 32 x 128 tiles
    "narrow": (9, 320, 576, E(0, 1, 31, 32, 33, 3, 65, 2, 7)),
    # few rows, over 512 MiB of weights: 32 x 256 tiles
    "streaming": (70, 1984, 2112, E(0, 40, 32, 1) + [11 + (5 * e) % 17 for e in range(66)]),
    # up projection on 128-row tiles (wide output), down projection on 32 x 128 ones
    "mid_narrow": (20, 192, 3136, E(0, 1, 127, 128, 129, 33, 2) + [30] * 13),
    # the same with more rows
    "mid_narrow_rows": (20, 192, 3136, E(0, 1, 63, 64, 65, 127, 128, 129, 257, 400) + [60] * 10),
    # up projection on 64-row tiles
    "mid64": (12, 320, 2112, E(0, 1, 63, 64, 65, 127, 128, 129, 200, 33, 31, 150)),
    # 128-row tiles both ways
    "mid": (16, 2112, 2240, E(0, 1, 127, 128, 129, 255, 256, 257, 300) + [64] * 7),
    # 288-row tiles both ways, with and without their extra block
    "fat": (16, 2496, 2560, E(288, 257, 256, 289, 0, 1, 31, 32, 33, 575, 576, 577, 512, 534, 490, 255)),
    # 288-row tiles up, 32 x 128 ones down
    "fat_narrow": (4, 256, 10240, E(288, 1, 577, 300)),
}

# the tiles of the up and down projection that each case is there for
TILES = {"narrow": ("32x128", "32x128"), "streaming": ("32x256", "32x256"), "mid_narrow": ("128x128", "32x128"),
         "mid_narrow_rows": ("128x128", "32x128"), "mid64": ("64x128", "32x128"), "mid": ("128x128", "128x128"),
         "fat": ("288x256", "288x256"), "fat_narrow": ("288x256", "32x128")}


def kernels(f):
    """The names of the kernels f enqueues."""
    lib, cap = abi.load(), 8
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(cap)]
    for e in ev:
        e.record()                                 # creates the event's handle
    handles, names = (ctypes.c_void_p * cap)(*[e.cuda_event for e in ev]), (ctypes.c_char_p * cap)()
    assert lib.dmoe_trace_begin(handles, names, cap) == 0
    f()
    return [names[i].decode() for i in range(lib.dmoe_trace_end())]


def close(got, ref, name):
    lim = 2e-2 * (ref.abs() + ref.square().mean().sqrt())
    bad = (got.double() - ref).abs() > lim + 1e-30
    assert not bool(bad.any()), f"{name}: {int(bad.sum())} of {bad.numel()} elements off"


@pytest.mark.parametrize("name", list(CASES))
def test_row_tile_shapes(name):
    N, D, H, counts = CASES[name]
    dev, g = torch.device("cuda:0"), torch.Generator(device="cuda").manual_seed(len(name))
    rows, P = sum(counts), sum(counts) + 5
    rn = lambda *s, sc=1.0: (torch.randn(*s, generator=g, device=dev) * sc).to(torch.bfloat16)
    dims = abi.make_dims(P, D, H, 1, N, 1, "bf16", "gelu")
    offs = torch.tensor([0] + counts, dtype=torch.int32).cumsum(0).to(torch.int32)
    W1, b1, W2, b2 = rn(N, H, D, sc=D ** -0.5), rn(N, H), rn(N, D, H, sc=H ** -0.5), rn(N, D)
    x, dy = rn(P, D), rn(P, D)
    ws = torch.full((abi.ffn_workspace_bytes(dims) + 256,), 255, dtype=torch.uint8, device=dev)   # 256 past its end
    nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device=dev)
    h, a, y, dh, dx = nan(P, H), nan(P, H), nan(P, D), nan(P, H), nan(P, D)
    dW1, db1, dW2, db2 = (torch.full_like(v, 7.0) for v in (W1, b1, W2, b2))
    off, cnt = offs.to(dev), torch.tensor(counts, dtype=torch.int32, device=dev)
    ran = kernels(lambda: abi.dmoe_expert_ffn_fwd(dims, off, x, W1, b1, W2, b2, h, a, y, ws))
    gemms = [n for n in ran if n.startswith("grouped_gemm2")]
    assert [any(f",{t}," in n for n in gemms[i:i + 1]) for i, t in enumerate(TILES[name])] == [True, True], gemms
    h2, a2, y2 = nan(P, H), nan(P, H), nan(P, D)
    abi.dmoe_expert_ffn_fwd_noalloc(dims, off, x, W1, b1, W2, b2, h2, a2, y2)
    abi.dmoe_expert_ffn_bwd(dims, off, cnt, x, h, a, dy, W1, W2, dh, dx, dW1, db1, dW2, db2, ws)
    hr, ar, dxr = nan(P, H), nan(P, H), nan(P, D)
    rW1, rb1, rW2, rb2 = (torch.full_like(v, 7.0) for v in (W1, b1, W2, b2))
    abi.dmoe_expert_ffn_bwd_recompute(dims, off, cnt, x, W1, b1, W2, dy, hr, ar, dxr, rW1, rb1, rW2, rb2, ws)
    torch.cuda.synchronize()
    assert bool((ws[-256:] == 255).all())
    for t in (h, a, y, dh, dx):
        assert bool(t[rows:].isnan().all()), f"{name}: rows past the last expert were written"
    for u, v in ((h, h2), (a, a2), (y, y2), (dx, dxr)):
        assert torch.equal(u[:rows], v[:rows]), name
    for u, v in ((dW1, rW1), (db1, rb1), (dW2, rW2), (db2, rb2)):
        assert torch.equal(u, v), name
    for e in range(N):
        s = slice(int(offs[e]), int(offs[e + 1]))
        if counts[e] == 0:
            assert all(bool((t[e] == 7.0).all()) for t in (dW1, db1, dW2, db2)), (name, e)
            continue
        w1, w2 = W1[e].double(), W2[e].double()
        z = x[s].double() @ w1.t() + b1[e].double()
        close(h[s], z, f"{name} expert {e} h")
        z = h[s].double()
        close(a[s], 0.5 * z * (1 + torch.erf(z * 0.5 ** 0.5)), f"{name} expert {e} a")
        close(y[s], a[s].double() @ w2.t() + b2[e].double(), f"{name} expert {e} y")
        da = 0.5 * (1 + torch.erf(z * 0.5 ** 0.5)) + z * torch.exp(-0.5 * z * z) * (2 * torch.pi) ** -0.5
        close(dh[s], (dy[s].double() @ w2) * da, f"{name} expert {e} dh")
        close(dx[s], dh[s].double() @ w1, f"{name} expert {e} dx")
        close(dW1[e], dh[s].double().t() @ x[s].double(), f"{name} expert {e} dW1")
        close(dW2[e], dy[s].double().t() @ a[s].double(), f"{name} expert {e} dW2")
