"""The two gate routes against the definition and against each other.

Exact route (fp64 matrix products, a wave per token selecting): gate columns at the edges
of the 16-column tiles and of the 64 lanes, ragged token counts, tied scores and totals
(small integers: every score is exact), scores of very different magnitude and sparse alive
sets with TopK among the alive experts (every cell is then ranked), there also with scores
that rise along the grid and that are all equal.  The reference ranks
every cell in fp64 by (alive first, total desc, flat index asc).

Certified route (bf16 matrix products plus recomputation of the rejected tokens): sizes
above the line where it is taken, which the launch trace confirms, for each column-block count
(1 to 3), wave count (one, and two from d_model 2048 on) and alive mode, against the exact route
on the same inputs (DMOE_FLAG_GATE_EXACT): the same experts in the same order, and weights
within the error the score bound allows (a few fp32 ulp).  The same with tokens that the
certificate has to reject, more of them than blocks that take the queue."""
import ctypes

import pytest
import torch

from paper_2002_04013_amd import abi

pytestmark = pytest.mark.gpu


def gate(dims, x, Wg, bg, alive, T, k, dM):
    dev = x.device
    idx = torch.full((T, k), -1, dtype=torch.int32, device=dev)
    w, g = (torch.full((T, k), -1.0, device=dev) for _ in range(2))
    sc = torch.empty((T, dM), device=dev)
    ws = torch.empty(abi.workspace_bytes(dims), dtype=torch.uint8, device=dev)
    abi.dmoe_gate_topk(dims, x, Wg, bg, alive, idx, w, g, sc, ws)
    torch.cuda.synchronize()
    return idx.cpu().long(), w.cpu(), g.cpu(), sc.cpu()


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


def reference(x, Wg, bg, alive, d, M, k, alive_first):
    S = x.double().cpu() @ Wg.double().cpu().t() + bg.double().cpu()
    dec = S.float().double().view(-1, d, M)
    tot = dec[:, 0]
    for i in range(1, d):
        tot = (tot[:, :, None] + dec[:, i][:, None, :]).reshape(tot.shape[0], -1)
    key = tot.clone()
    order = torch.sort(key, dim=1, descending=True, stable=True)[1]
    if alive_first:                       # stable: alive ones first, each kind in order
        dead = (alive.cpu()[order] == 0).to(torch.uint8)
        order = order.gather(1, torch.sort(dead, dim=1, stable=True)[1])
    idx = order[:, :k]
    g = sum(S.gather(1, idx // M ** (d - 1 - i) % M + i * M) for i in range(d))
    live = alive.cpu()[idx] != 0
    ex = torch.where(live, torch.exp(g - torch.where(live, g, torch.full_like(g, -1e300)).max(1, keepdim=True)[0]),
                     torch.zeros_like(g))
    w = torch.where(live, ex / ex.sum(1, keepdim=True), torch.zeros_like(ex))
    return S, idx, g, w


# dtype, T, D, d, M, k, inputs, p_alive, alive_first
EXACT = [
    ("f32", 1, 64, 1, 2, 1, "normal", 1.0, False), ("f32", 31, 64, 1, 16, 8, "ties", 1.0, False),
    ("f32", 33, 192, 1, 17, 5, "normal", 0.8, False), ("f32", 100, 128, 1, 128, 8, "ties", 0.9, False),
    ("f32", 64, 64, 2, 4, 8, "ties", 0.5, True), ("f32", 70, 256, 4, 3, 8, "ties", 0.6, True),
    ("f32", 65, 64, 4, 11, 8, "normal", 0.3, True), ("f32", 40, 64, 3, 5, 4, "span", 0.9, False),
    ("f32", 40, 64, 3, 5, 4, "span", 0.2, True), ("f32", 96, 1024, 2, 33, 4, "normal", 0.95, False),
    ("bf16", 130, 512, 2, 64, 8, "ties", 0.9, False), ("bf16", 63, 64, 2, 49, 8, "normal", 0.02, True),
    ("bf16", 200, 320, 3, 16, 4, "ties", 0.9, True), ("bf16", 77, 64, 2, 8, 3, "span", 0.9, False),
    ("bf16", 300, 128, 4, 8, 8, "ties", 0.9, False), ("bf16", 50, 2112, 3, 25, 8, "normal", 0.5, True),
    # few candidates for the tokens: a lane per token selects
    ("f32", 32801, 64, 2, 16, 4, "normal", 0.9, False), ("f32", 32768, 64, 2, 15, 3, "ties", 0.8, False),
    ("f32", 16385, 192, 1, 16, 1, "normal", 0.9, False), ("f32", 20000, 64, 2, 4, 4, "span", 0.9, False),
    ("f32", 16400, 1024, 2, 2, 4, "normal", 1.0, False), ("f32", 32800, 128, 4, 3, 4, "ties", 0.9, False),
    ("f32", 33, 64, 1, 2, 1, "normal", 0.5, False), ("f32", 2049, 64, 2, 2, 3, "ties", 0.9, False),
    ("f32", 9000, 64, 3, 3, 2, "span", 0.9, False),
    ("f32", 65537, 64, 2, 4, 8, "ties", 0.9, False), ("f32", 65600, 64, 1, 64, 4, "normal", 0.9, False),
    ("f32", 20, 64, 2, 40, 8, "rising", 0.2, True), ("bf16", 20, 64, 3, 25, 8, "rising", 0.003, True),
    ("f32", 20, 64, 2, 30, 8, "equal", 0.1, True), ("f32", 20, 64, 2, 64, 8, "ties", 0.05, True),
]


@pytest.mark.parametrize("dtype,T,D,d,M,k,inputs,p_alive,alive_first", EXACT)
def test_exact_route_matches_the_definition(dtype, T, D, d, M, k, inputs, p_alive, alive_first):
    gen = torch.Generator().manual_seed(T * 131 + D + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    dM, N = d * M, M ** d
    if inputs == "normal":
        x, Wg, bg = (torch.randn(*s, generator=gen) for s in ((T, D), (dM, D), (dM,)))
        Wg *= D ** -0.5
    else:                                 # small integers: exact scores, many of them equal
        x = torch.randint(-1, 2, (T, D), generator=gen).float()
        Wg = torch.randint(-1, 2, (dM, D), generator=gen).float() * (torch.rand(dM, D, generator=gen) < 8.0 / D)
        bg = torch.randint(-1, 2, (dM,), generator=gen).float()
        if inputs in ("rising", "equal"):  # each cell beats those before it; all scores 0
            Wg.zero_()
            bg = torch.arange(M).float().repeat(d) if inputs == "rising" else torch.zeros(dM)
            bg[:M * (d - 1)] *= 8.0
        if inputs == "span":              # one column of each dimension 2^30 times the others
            Wg[::M] *= 2.0 ** 30
    x, Wg, bg = x.to(dt).cuda(), Wg.to(dt).cuda(), bg.to(dt).cuda()
    alive = (torch.rand(N, generator=gen) < p_alive).to(torch.uint8)
    dims = abi.make_dims(T, D, 64, d, M, k, dtype, "relu", abi.DMOE_FLAG_ALIVE_TOPK if alive_first else 0)
    idx, w, g, sc = gate(dims, x, Wg, bg, alive.cuda(), T, k, dM)
    S, ridx, rg, rw = reference(x, Wg, bg, alive, d, M, k, alive_first)
    assert torch.equal(idx, ridx)
    assert torch.equal(sc, S.float()) or float((sc - S).abs().max()) <= 2.0 ** -23 * float(S.abs().max())
    assert float((g - rg).abs().max()) <= 2.0 ** -23 * float(rg.abs().max())
    assert float((w - rw).abs().max()) <= 2e-6       # fp32 exp and division of exact totals


@pytest.mark.parametrize("T,D,d,M,k,p_alive,alive_first", [
    # columns up to 32, one wave a block and two
    (44000, 64, 2, 4, 4, 0.9, False), (43001, 64, 1, 32, 8, 0.9, True), (33000, 2048, 2, 16, 4, 1.0, False),
    (40001, 2112, 2, 16, 8, 0.9, True),
    # narrow d_model, as many cells as are chosen or ranked
    (16400, 64, 2, 2, 4, 0.9, False), (12301, 64, 2, 2, 2, 0.9, True), (14001, 128, 1, 16, 1, 0.9, False),
    # up to 64
    (40000, 1024, 2, 32, 4, 0.95, False), (40000, 1024, 2, 32, 4, 0.9, True), (20000, 2112, 2, 17, 8, 0.9, False),
    (20000, 2048, 4, 11, 4, 0.9, True),
    # up to 96
    (30000, 1088, 3, 25, 4, 0.95, False), (50003, 1024, 2, 40, 8, 0.9, True), (16400, 2048, 2, 48, 8, 0.8, False),
    (16400, 2048, 2, 48, 4, 0.8, True),
])
def test_certified_route_matches_the_exact_one(T, D, d, M, k, p_alive, alive_first):
    g = torch.Generator(device="cuda").manual_seed(T)
    dM, N = d * M, M ** d
    x = torch.randn(T, D, generator=g, device="cuda").to(torch.bfloat16)
    Wg = (torch.randn(dM, D, generator=g, device="cuda") * D ** -0.5).to(torch.bfloat16)
    bg = torch.randn(dM, generator=g, device="cuda").to(torch.bfloat16)
    alive = (torch.rand(N, generator=g, device="cuda") < p_alive).to(torch.uint8)
    fl = abi.DMOE_FLAG_ALIVE_TOPK if alive_first else 0
    out = []
    ran = [kernels(lambda: out.append(gate(abi.make_dims(T, D, 64, d, M, k, "bf16", "relu", f), x, Wg, bg, alive, T, k, dM)))
           for f in (fl, fl | abi.DMOE_FLAG_GATE_EXACT)]
    assert any("gate_topk_mfma" in n for n in ran[0]) and ran[1] == ["gate_topk_f64"], ran
    assert torch.equal(out[0][0], out[1][0])
    # |score error| <= gamma_32 sum |x w| (about 4e-6 * 0.64 sqrt(D)); a weight moves by at most 2 w d times that
    lim = 4.1e-6 * float((x[:64].float().abs() @ Wg.float().abs().t()).max()) * 1.5 + 2.0 ** -22 * float(out[1][3].abs().max())
    assert float((out[0][3] - out[1][3]).abs().max()) <= lim
    assert float((out[0][2] - out[1][2]).abs().max()) <= d * lim
    assert float((out[0][1] - out[1][1]).abs().max()) <= 2 * d * lim + 1e-6


@pytest.mark.parametrize("inputs", ["ties", "near_ties", "span"])
@pytest.mark.parametrize("T,D,d,M,k,p_alive,alive_first", [
    (40000, 1024, 2, 16, 4, 0.9, False), (20000, 2048, 2, 32, 8, 0.9, False), (40000, 1024, 2, 30, 4, 0.7, True),
    (17000, 2112, 3, 25, 4, 0.9, True),
])
def test_certified_route_rejects(T, D, d, M, k, p_alive, alive_first, inputs):
    """Every third token is one the certificate cannot decide: equal gate rows (exact ties, the
    lower flat index first), rows that differ in the last bit of one weight, or scores that span
    more than 2^25.  Against the definition for a sample of tokens
    and against the exact route for all; the certified tokens between them stay as they are."""
    g = torch.Generator(device="cuda").manual_seed(T + M)
    dM, N = d * M, M ** d
    x = torch.randn(T, D, generator=g, device="cuda").to(torch.bfloat16)
    Wg = (torch.randn(dM, D, generator=g, device="cuda") * D ** -0.5).to(torch.bfloat16)
    bg = torch.randn(dM, generator=g, device="cuda").to(torch.bfloat16)
    alive = (torch.rand(N, generator=g, device="cuda") < p_alive).to(torch.uint8)
    third = torch.arange(0, T, 3, device="cuda")
    if inputs == "span":
        # column 0 of each dimension scores x[0] + 2^-34, and x[0] is 0 on those tokens
        Wg[::M], bg[::M] = 0, 0
        Wg[::M, 0], Wg[::M, 1] = 1.0, 2.0 ** -34
        x[:, 1], x[third, 0] = 1.0, 0.0
    else:
        # on those tokens x is 0 but for its first 64 values, where rows u and u + 1 agree
        keep = torch.zeros(D, dtype=torch.bool, device="cuda")
        keep[:64] = True
        x[third] = torch.where(keep, x[third], torch.zeros_like(x[third]))
        for i in range(d):
            for u in range(0, M - 1, 2):
                Wg[i * M + u + 1, :64], bg[i * M + u + 1] = Wg[i * M + u, :64], bg[i * M + u]
                if inputs == "near_ties":
                    Wg[i * M + u + 1, 7] = Wg[i * M + u, 7] * (1 + 2.0 ** -7)
        if inputs == "near_ties":
            x[third, 7] = 2.0 ** -14
    fl = abi.DMOE_FLAG_ALIVE_TOPK if alive_first else 0
    dims = abi.make_dims(T, D, 64, d, M, k, "bf16", "relu", fl)
    out = []
    assert any("gate_topk_mfma" in n for n in kernels(lambda: out.append(gate(dims, x, Wg, bg, alive, T, k, dM))))
    out.append(gate(abi.make_dims(T, D, 64, d, M, k, "bf16", "relu", fl | abi.DMOE_FLAG_GATE_EXACT), x, Wg, bg, alive, T, k,
                    dM))
    assert torch.equal(out[0][0], out[1][0])
    # the tokens were rejected: their scores are the exact route's, which certified ones rarely are
    rec = (out[0][3] == out[1][3]).all(1)
    assert int(rec[third.cpu()].sum()) > 1024 and bool(rec[third.cpu()].all())
    n = 600
    _, ridx, _, rw = reference(x[:n], Wg, bg, alive, d, M, k, alive_first)
    assert torch.equal(out[0][0][:n], ridx)
    assert float((out[0][1][:n] - rw).abs().max()) <= 1e-4


@pytest.mark.parametrize("dtype,T,D,d,M,k,p_alive,alive_first", [
    ("f32", 65, 64, 2, 6, 4, 1.0, False), ("f32", 40, 64, 3, 5, 8, 0.6, True), ("f32", 50, 128, 1, 100, 8, 0.9, False),
    ("bf16", 77, 64, 2, 9, 4, 0.9, False), ("bf16", 130, 128, 2, 60, 8, 0.6, True),
    ("bf16", 40000, 1024, 2, 16, 4, 0.9, False), ("bf16", 40000, 1024, 2, 32, 4, 0.6, True),   # certified
])
def test_non_finite_scores(dtype, T, D, d, M, k, p_alive, alive_first):
    """Two gate columns whose weights are NaN: every token is routed among the others, with
    finite weights.  Tokens with infinities or a NaN of their own: valid expert ids."""
    gen = torch.Generator().manual_seed(T + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    dM, N, n = d * M, M ** d, min(T, 2000)
    x, Wg, bg = (torch.randn(*s, generator=gen) for s in ((T, D), (dM, D), (dM,)))
    Wg *= D ** -0.5
    alive = (torch.rand(N, generator=gen) < p_alive).to(torch.uint8)
    Wg[1], Wg[(d - 1) * M + 2, 3] = float("nan"), float("nan")
    x[5, 1], x[7, 1], x[9, 2], x[11, :] = float("inf"), float("nan"), -float("inf"), float("inf")
    x, Wg, bg = x.to(dt), Wg.to(dt), bg.to(dt)
    dims = abi.make_dims(T, D, 64, d, M, k, dtype, "relu", abi.DMOE_FLAG_ALIVE_TOPK if alive_first else 0)
    idx, w, g, _ = gate(dims, x.cuda(), Wg.cuda(), bg.cuda(), alive.cuda(), T, k, dM)
    assert int(idx.min()) >= 0 and int(idx.max()) < N
    keep = torch.ones(T, dtype=torch.bool)
    keep[[5, 7, 9, 11]] = False
    assert bool(w[keep].isfinite().all()) and bool(g[keep].isfinite().all())
    keep = keep[:n]
    S = x[:n].double() @ Wg.double().t() + bg.double()      # NaN columns below every other
    S = torch.where(S.isnan(), torch.full_like(S, -1e30), S)
    _, ridx, rg, rw = reference(S[keep], torch.eye(dM), torch.zeros(dM), alive, d, M, k, alive_first)
    assert torch.equal(idx[:n][keep], ridx)
    assert float((w[:n][keep] - rw).abs().max()) <= 1e-4    # bf16 score bound of the certified route
