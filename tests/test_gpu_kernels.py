"""Small GPU checks of kernels and dispatch branches at the sizes where they can go wrong."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

REL = 1  # CB_LAMBDA_RELATIVE
UNPEN = 2  # CB_RIDGE_BIAS_UNPENALIZED


@pytest.fixture(scope="module")
def cb():
    import paper_2609_00891_amd as lib
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return lib


def _moments(n, P, dt, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((n, 3 * P, P)) * np.exp(rng.standard_normal(P))
    x[:, :, -1] = 1.0
    y = rng.standard_normal((n, 3 * P, dt))
    G = np.matmul(x.transpose(0, 2, 1), x).astype(np.float32)
    G = np.triu(G) + np.triu(G, 1).transpose(0, 2, 1)
    return np.ascontiguousarray(G), np.matmul(x.transpose(0, 2, 1), y).astype(np.float32)


def _relF(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# The narrow solver: every block count of both widths, more systems than fit the chip at once and a single one,
# both bias conventions.  fp64 inside, so only the final rounding to fp32 (2^-24 relative per element) is seen: 1e-6.
@pytest.mark.parametrize("n", [1, 600])
@pytest.mark.parametrize("dt", [64, 96, 128])
@pytest.mark.parametrize("ds", [64, 96, 128])
def test_narrow_solve_widths(cb, ds, dt, n):
    import oracle
    G, C = _moments(min(n, 5), ds + 1, dt, ds + dt)
    reps = -(-n // G.shape[0])
    Gd, Cd = (torch.from_numpy(np.tile(a, (reps, 1, 1))[:n]).cuda() for a in (G, C))
    for flags in (REL, REL | UNPEN, 0):
        maps, info = torch.full_like(Cd, 7.0), torch.full((n,), -1, dtype=torch.int32, device="cuda")
        cb.cb_ridge_solve(Gd, Cd, 1e-2, flags, maps, info)
        W, io = oracle.ridge_solve(G.astype(np.float64), C.astype(np.float64), 1e-2, relative=bool(flags & REL),
                                   bias_unpenalized=bool(flags & UNPEN))
        assert (io == 0).all() and (info.cpu().numpy() == 0).all()
        got = maps.double().cpu().numpy()
        for m in range(n):
            assert _relF(got[m], W[m % G.shape[0]]) < 1e-6, (ds, dt, n, flags, m)


# The first pivot that fails, inside a 16-wide block, at its edges and on the bias row; the other systems of the
# batch are untouched by it.
@pytest.mark.parametrize("ds", [64, 96, 128])
def test_narrow_solve_failing_pivots(cb, ds):
    import oracle
    dt = 64
    at = sorted({0, 1, 15, 16, 17, 31, 47, 48, ds - 16, ds - 1, ds})
    G, C = _moments(len(at) + 1, ds + 1, dt, 11)
    for m, k in enumerate(at):
        G[m, k, k] = -1.0
    G[0, 5, 5] = np.nan                                    # behind the first failing pivot: still reported at 0
    Gd, Cd = torch.from_numpy(G).cuda(), torch.from_numpy(C).cuda()
    maps, info = torch.full_like(Cd, 7.0), torch.full((len(at) + 1,), -1, dtype=torch.int32, device="cuda")
    cb.cb_ridge_solve(Gd, Cd, 1e-3, 0, maps, info)
    assert info.cpu().tolist() == [k + 1 for k in at] + [0]
    assert (maps[:-1] == 0).all()
    W, _ = oracle.ridge_solve(G[-1:].astype(np.float64), C[-1:].astype(np.float64), 1e-3, relative=False)
    assert _relF(maps[-1].double().cpu().numpy(), W[0]) < 1e-6


# The wide solver: the first width past the narrow one, panels that end ragged, one past a multiple of 128 (the bias
# kept as a column of its own) and on it, one and two panels short of 1025; a workspace of exactly one system (every
# system a batch of its own), one of two and a half, and the fixed scratch; all against the oracle.
@pytest.mark.parametrize("P", [130, 144, 161, 200, 256, 257, 300, 385, 400, 1025])
@pytest.mark.parametrize("dt", [64, 96, 128])
def test_wide_solve_shapes(cb, P, dt):
    import oracle
    if P > 400 and dt != 128:
        pytest.skip("one width is enough at this size")
    n = 3
    G, C = _moments(n, P, dt, P + dt)
    # the middle system fails at P // 2 + 1: its diagonal there is -tr / P, past the ridge of tr / (100 P)
    G[1, P // 2, P // 2] = -np.trace(G[1]) / P
    W, io = oracle.ridge_solve(G.astype(np.float64), C.astype(np.float64), 1e-2, relative=True, bias_unpenalized=True)
    assert io.tolist() == [0, P // 2 + 1, 0]
    Gd, Cd = torch.from_numpy(G).cuda(), torch.from_numpy(C).cuda()
    one = cb.cb_ridge_solve_workspace_bytes(P, dt, 1)
    assert one == 8 * (P * P + P * dt)
    for ws_bytes in (one, 2 * one + one // 2, None):
        maps, info = torch.full_like(Cd, 7.0), torch.full((n,), -1, dtype=torch.int32, device="cuda")
        if ws_bytes is None:
            cb.cb_ridge_solve_noalloc(Gd, Cd, 1e-2, REL | UNPEN, maps, info)
        else:
            # exactly the bytes asked for, with guard values behind them
            buf = torch.full((ws_bytes // 8 + 64,), 3.0, dtype=torch.float64, device="cuda")
            cb.cb_ridge_solve_ws(Gd, Cd, 1e-2, REL | UNPEN, maps, info, buf[:ws_bytes // 8])
            assert (buf[ws_bytes // 8:] == 3.0).all()
        assert info.cpu().tolist() == io.tolist()
        assert (maps[1] == 0).all()
        for m in (0, 2):
            assert _relF(maps[m].double().cpu().numpy(), W[m]) < 1e-6, (P, dt, ws_bytes, m)


# Centered systems: a width that is a multiple of 128 (no bias column in the system) and one past it, whose last
# feature takes the bias column's place.
@pytest.mark.parametrize("dx", [256, 257, 330])
def test_wide_solve_centered_shapes(cb, dx):
    import oracle
    n, dt = 2, 96
    G, C = _moments(n, dx, dt, dx)
    rng = np.random.default_rng(dx)
    sums = np.concatenate([np.full((n, 1), 50.0), 20 * rng.standard_normal((n, dx + dt))], axis=1)
    W, io = oracle.ridge_solve_centered(sums, G.astype(np.float64), C.astype(np.float64), 1e-3, relative=True)
    ws = torch.empty(cb.cb_ridge_solve_workspace_bytes(dx, dt, n), dtype=torch.uint8, device="cuda")
    maps = torch.full((n, dx + 1, dt), 7.0, device="cuda")
    info = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cb.cb_ridge_solve_centered_ws(torch.from_numpy(sums).cuda(), torch.from_numpy(G).cuda(), torch.from_numpy(C).cuda(),
                                  1e-3, REL, maps, info, ws)
    assert (info.cpu().numpy() == 0).all() and (io == 0).all()
    for m in range(n):
        assert _relF(maps[m].double().cpu().numpy(), W[m]) < 1e-6


# Probe R^2 for every width pair against the same formula in fp64.  The kernel forms A W with fp32 sums of d_s
# products: each element is off by at most d_s 2^-24 sum |A_ik W_kj|, hence the bound on tr(W^T A W) below.
@pytest.mark.parametrize("dt", [64, 96, 128])
@pytest.mark.parametrize("ds", [64, 96, 128])
def test_probe_r2_widths(cb, ds, dt):
    n = 5
    rng = np.random.default_rng(ds * dt)
    A, B = _moments(n, ds, dt, ds + dt)
    W = (rng.standard_normal((n, ds + 1, dt)) / ds).astype(np.float32)
    sums = np.concatenate([np.full((n, 1), 3.0 * ds), rng.standard_normal((n, ds + dt))], axis=1)
    sq = np.abs(rng.standard_normal((n, ds + dt))) * 1e4
    sums[4] = 0.0                                          # no data: R^2 is 0
    sq[3] = 0.0                                            # no variance: R^2 is 0
    r2 = torch.full((n,), 9.0, dtype=torch.float64, device="cuda")
    cb.cb_probe_r2(*(torch.from_numpy(x).cuda() for x in (sums, sq, A, B, W)), r2)
    got = r2.cpu().numpy()
    for m in range(3):
        w, a = W[m, :ds].astype(np.float64), A[m].astype(np.float64)
        tss = (sq[m, ds:] - sums[m, 1 + ds:] ** 2 / sums[m, 0]).sum()
        rss = tss - 2 * (w * B[m]).sum() + (w * (a @ w)).sum()
        bound = ds * 2.0 ** -24 * (np.abs(w) * (np.abs(a) @ np.abs(w))).sum() / tss
        assert abs(got[m] - (1 - rss / tss)) <= bound + 1e-12
    assert got[3] == 0.0 and got[4] == 0.0


# Token tiles of a call cut into chunks by size: one chunk per item, several, a last chunk shorter than the others, and
# tiles that end inside a sequence; 3 target layers of 2 heads leave a chip-filling number of chunks, 300 maps do not.
# fp32 sums of exact products with the weight in two bf16 terms: 1e-5 is ten times what the largest call shows.
@pytest.mark.parametrize("layers,seqs,T", [(3, 1, 31), (3, 1, 2048), (3, 5, 333), (75, 1, 1000), (75, 3, 700)])
@pytest.mark.parametrize("centered", [False, True])
def test_stats_chunks(cb, layers, seqs, T, centered):
    H, d = 2, 64
    rows = [(l, h, z, l % 5, h, l * H + h) for l in range(layers) for z in range(2) for h in range(H)]
    names = ("tgt_layer", "tgt_head", "kv", "src_layer", "src_head", "weight_row")
    hm = {k: np.asarray(v, dtype=np.int32) for k, v in zip(names, zip(*rows))}
    n, g = len(rows), torch.Generator(device="cuda").manual_seed(seqs * T)
    src = torch.randn((5, 2, seqs, H, T, d), generator=g, device="cuda").bfloat16()
    tgt = torch.randn((layers, 2, seqs, H, T, d), generator=g, device="cuda").bfloat16()
    w = torch.rand((layers * H, seqs * T), generator=g, device="cuda")
    plan = cb.cb_plan_create(hm, src, tgt, seqs * T)
    ref = []
    for l, h, z, sl, sh, wr in rows:
        x = src[sl, z, :, sh].reshape(-1, d).double()
        y = tgt[l, z, :, h].reshape(-1, d).double()
        ww = w[wr].double()[:, None]
        if centered:
            x, y = x - (ww * x).sum(0) / ww.sum(), y - (ww * y).sum(0) / ww.sum()
        else:
            x = torch.cat([x, torch.ones_like(x[:, :1])], dim=1)
        ref.append(((x * ww).t() @ x, (x * ww).t() @ y))
    P = d if centered else d + 1
    G, C = torch.ones((n, P, P), device="cuda"), torch.ones((n, P, d), device="cuda")
    if centered:
        sums = torch.zeros((n, 1 + 2 * d), dtype=torch.float64, device="cuda")
        cb.cb_stats_means(plan, src, tgt, w, sums)
        cb.cb_stats_accumulate_centered(plan, src, tgt, w, sums, G, C)
    else:
        cb.cb_stats_accumulate(plan, src, tgt, w, G, C)
    assert torch.equal(G, G.transpose(1, 2))
    for m, (rg, rc) in enumerate(ref):
        for got, want in ((G[m], rg + 1), (C[m], rc + 1)):           # added to what was there
            assert float((got.double() - want).norm() / want.norm()) < 1e-5, (m, layers, seqs, T)


# Token tiles of the single-layer application: one token, the edges of a 32-token sub-block, several tiles and more
# than the 8192 tokens of one, a source block of two maps and one of a single map; the maps at an address that is only
# 4-byte aligned.  An element is the fp64 value rounded once, up to one bf16 ulp where the fp32 sum (coefficients as two
# bf16 terms, 2^-17 of the sum of |x W|, far below 1e-4 of the outputs' RMS) falls on the other side of a tie.
@pytest.mark.parametrize("T", [1, 31, 33, 500, 8225])
@pytest.mark.parametrize("ds,dt", [(64, 128), (96, 64), (128, 96)])
def test_apply_token_tiles(cb, ds, dt, T):
    names = ("tgt_layer", "tgt_head", "kv", "src_layer", "src_head", "weight_row")
    rows = [(0, 0, 0, 0, 0, 0), (1, 0, 0, 0, 0, 0), (0, 0, 1, 1, 0, 0)]      # two maps of one block, one alone
    hm = {k: np.asarray(v, dtype=np.int32) for k, v in zip(names, zip(*rows))}
    g = torch.Generator(device="cuda").manual_seed(T)
    src = torch.randn((2, 2, 1, 1, T, ds), generator=g, device="cuda").bfloat16()
    flat = torch.randn(3 * (ds + 1) * dt + 1, generator=g, device="cuda") / ds ** 0.5
    maps = flat[1:].view(3, ds + 1, dt)
    out = torch.full((2, 2, 1, 1, T + 1, dt), 5.0, dtype=torch.bfloat16, device="cuda")
    plan = cb.cb_plan_create(hm, src, out, T)
    cb.cb_apply(plan, maps, src, out[:, :, :, :, :T])
    for m, (tl, _, z, sl, _, _) in enumerate(rows):
        ref = src[sl, z, 0, 0].double() @ maps[m, :-1].double() + maps[m, -1].double()
        got = out[tl, z, 0, 0, :T].double()
        bound = ref.abs() * 2.0 ** -8 + 1e-4 * ref.square().mean().sqrt()
        assert bool(((got - ref).abs() <= bound).all()), (m, ds, dt, T)
    assert bool((out[:, :, :, :, T:] == 5.0).all()) and bool((out[1, 1] == 5.0).all())


# Multi-layer moments of a call long enough to be added into G and C twice (every 32,736 rows) and of the shortest
# ones, k with a half-used task rectangle among them; what was in G and C stays.  1e-5: fp32 sums over 32,736 rows.
@pytest.mark.parametrize("k,T,stride", [(2, 33001, 1), (3, 17, 4), (1, 5, 1), (5, 131, 2)])
@pytest.mark.parametrize("centered", [False, True])
def test_multi_stats_flushes(cb, k, T, stride, centered):
    d, L, n = 128, 6, 2
    hm = dict(tgt_layer=[0, 0], tgt_head=[0, 0], kv=[0, 1], src_layers=[[(2 * j + m) % L for j in range(k)] for m in range(n)],
              src_head=[0, 0], weight_row=[0, 1])
    if k == 5:
        hm["src_layers"] = [[0, 1, 2, 3, 4], [5, 4, 3, 2, 1]]
    g = torch.Generator(device="cuda").manual_seed(T)
    src = torch.randn((L, 2, 1, 1, T, d), generator=g, device="cuda").bfloat16()
    tgt = torch.randn((1, 2, 1, 1, T, d), generator=g, device="cuda").bfloat16()
    w = torch.rand((2, T), generator=g, device="cuda")
    plan = cb.cb_plan_create_multi(hm, src, tgt, stride)
    P = k * d + (0 if centered else 1)
    G, C = torch.ones((n, P, P), device="cuda"), torch.ones((n, P, d), device="cuda")
    if centered:
        sums = torch.zeros((n, 1 + P + d), dtype=torch.float64, device="cuda")
        cb.cb_stats_means(plan, src, tgt, w, sums)
        cb.cb_stats_accumulate_centered(plan, src, tgt, w, sums, G, C)
    else:
        cb.cb_stats_accumulate(plan, src, tgt, w, G, C)
    assert torch.equal(G, G.transpose(1, 2))
    for m in range(n):
        x = torch.cat([src[j, m, 0, 0, ::stride].double() for j in hm["src_layers"][m]], dim=1)
        y, ww = tgt[0, m, 0, 0, ::stride].double(), w[m, ::stride].double()[:, None]
        if centered:
            x, y = x - (ww * x).sum(0) / ww.sum(), y - (ww * y).sum(0) / ww.sum()
        else:
            x = torch.cat([x, torch.ones_like(x[:, :1])], dim=1)
        for got, want in ((G[m], (x * ww).t() @ x + 1), (C[m], (x * ww).t() @ y + 1)):
            assert float((got.double() - want).norm() / want.norm()) < 1e-5


# Plans whose maps share target rows (every target layer with every source layer), their units in consecutive runs per
# XCD: fewer units than XCDs, counts that are no multiple of eight, one chunk and several.  1e-5 as for the chunks.
@pytest.mark.parametrize("Lt,Ls,H,T", [(2, 1, 1, 33), (1, 3, 1, 500), (3, 5, 1, 2100), (5, 7, 2, 130)])
@pytest.mark.parametrize("d", [64, 128])
def test_stats_shared_targets(cb, d, Lt, Ls, H, T):
    rows = [(l, h, z, s, h, l * H + h) for l in range(Lt) for s in range(Ls) for z in range(2) for h in range(H)]
    rows += rows[:1]                                                    # one map twice: shared targets at Ls = 1 too
    names = ("tgt_layer", "tgt_head", "kv", "src_layer", "src_head", "weight_row")
    hm = {k: np.asarray(v, dtype=np.int32) for k, v in zip(names, zip(*rows))}
    n, g = len(rows), torch.Generator(device="cuda").manual_seed(T)
    src = torch.randn((Ls, 2, 2, H, T, d), generator=g, device="cuda").bfloat16()
    tgt = torch.randn((Lt, 2, 2, H, T, d), generator=g, device="cuda").bfloat16()
    w = torch.rand((Lt * H, 2 * T), generator=g, device="cuda")
    plan = cb.cb_plan_create(hm, src, tgt, 2 * T)
    G, C = torch.zeros((n, d + 1, d + 1), device="cuda"), torch.zeros((n, d + 1, d), device="cuda")
    A, B = torch.zeros((n, d, d), device="cuda"), torch.zeros((n, d, d), device="cuda")
    sums = torch.zeros((n, 1 + 2 * d), dtype=torch.float64, device="cuda")
    sq = torch.zeros((n, 2 * d), dtype=torch.float64, device="cuda")
    cb.cb_stats_accumulate(plan, src, tgt, w, G, C)
    cb.cb_stats_means(plan, src, tgt, w, sums, sq=sq)
    cb.cb_stats_accumulate_centered(plan, src, tgt, w, sums, A, B)
    for m, (l, h, z, s, _, wr) in enumerate(rows):
        x, y, ww = src[s, z, :, h].reshape(-1, d).double(), tgt[l, z, :, h].reshape(-1, d).double(), w[wr].double()[:, None]
        x1, xy = torch.cat([x, torch.ones_like(x[:, :1])], dim=1), torch.cat([x, y], dim=1)
        xc, yc = x - (ww * x).sum(0) / ww.sum(), y - (ww * y).sum(0) / ww.sum()
        s1 = torch.cat([ww.sum(0), (ww * xy).sum(0)])
        for got, want in ((G, (x1 * ww).t() @ x1), (C, (x1 * ww).t() @ y), (A, (xc * ww).t() @ xc), (B, (xc * ww).t() @ yc),
                          (sums, s1), (sq, (ww * xy * xy).sum(0))):
            assert float((got[m].double() - want).norm() / want.norm()) < 1e-5, (m, d, Lt, Ls, H, T)


# Systems that fail at their bias pivot alone (one column past a multiple of 128), many of them between good ones: every
# workgroup of a failing system writes zeros, whichever of them reports the pivot first.
@pytest.mark.parametrize("P", [257, 513])
def test_wide_solve_bias_pivots(cb, P):
    dt, n = 128, 96
    G, C = _moments(2, P, dt, P)
    G[0, -1, -1] = -1.0
    Gd, Cd = (torch.from_numpy(a).cuda().repeat(n // 2, 1, 1) for a in (G, C))
    ws = torch.empty(cb.cb_ridge_solve_workspace_bytes(P, dt, n), dtype=torch.uint8, device="cuda")
    good = None
    for _ in range(20):
        maps, info = torch.full_like(Cd, 7.0), torch.full((n,), -1, dtype=torch.int32, device="cuda")
        cb.cb_ridge_solve_ws(Gd, Cd, 1e-3, 0, maps, info, ws)
        assert info.cpu().tolist() == [P, 0] * (n // 2)
        assert bool((maps[0::2] == 0).all())
        good = maps[1].clone() if good is None else good
        assert bool((maps[1::2] == good).all())


# In place, maps = C: every column of C is read before the coefficients take its place.
@pytest.mark.parametrize("P", [65, 129, 257, 300, 513])
def test_solve_in_place(cb, P):
    dt, n = 128, 40
    G, C = _moments(2, P, dt, P)
    Gd, Cd = (torch.from_numpy(a).cuda().repeat(n // 2, 1, 1) for a in (G, C))
    info = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(cb.cb_ridge_solve_workspace_bytes(P, dt, n), 8), dtype=torch.uint8, device="cuda")
    maps, both = torch.empty_like(Cd), Cd.clone()
    cb.cb_ridge_solve_ws(Gd, Cd, 1e-2, REL | UNPEN, maps, info, ws)
    cb.cb_ridge_solve_ws(Gd, both, 1e-2, REL | UNPEN, both, info, ws)
    assert torch.equal(maps, both) and bool((info == 0).all())


# Batches that fill the chip: the back substitution takes a system per workgroup (up to six panels) or 16 right-hand
# sides per workgroup.  Ragged last panels and the bias column, a system that fails inside and one at its bias pivot.
@pytest.mark.parametrize("n", [255, 256])
@pytest.mark.parametrize("P,dt", [(130, 64), (161, 128), (257, 96), (300, 128), (769, 64), (770, 64)])
def test_wide_solve_many_systems(cb, P, dt, n):
    import oracle
    G, C = _moments(4, P, dt, P + dt)
    G[1, P // 2, P // 2] = -1.0
    G[2, -1, -1] = -1.0
    W, io = oracle.ridge_solve(G.astype(np.float64), C.astype(np.float64), 1e-3, relative=False)
    assert io.tolist() == [0, P // 2 + 1, P, 0]
    Gd, Cd = (torch.from_numpy(a).cuda().repeat(-(-n // 4), 1, 1)[:n].contiguous() for a in (G, C))
    maps, info = torch.full_like(Cd, 7.0), torch.full((n,), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(cb.cb_ridge_solve_workspace_bytes(P, dt, n), dtype=torch.uint8, device="cuda")
    cb.cb_ridge_solve_ws(Gd, Cd, 1e-3, 0, maps, info, ws)
    assert info.cpu().tolist() == [int(io[m % 4]) for m in range(n)]
    for k in range(4):
        assert bool((maps[k::4] == maps[k]).all()), (P, dt, n, k)
    assert bool((maps[1:3] == 0).all())
    for k in (0, 3):
        assert _relF(maps[k].double().cpu().numpy(), W[k]) < 1e-6


@pytest.mark.parametrize("dx", [256, 257, 330])
def test_wide_solve_many_centered(cb, dx):
    import oracle
    n, dt = 256, 96
    G, C = _moments(2, dx, dt, dx)
    rng = np.random.default_rng(dx)
    sums = np.concatenate([np.full((2, 1), 50.0), 20 * rng.standard_normal((2, dx + dt))], axis=1)
    sums[1] = 0.0                                          # no data: means of zero
    W, io = oracle.ridge_solve_centered(sums, G.astype(np.float64), C.astype(np.float64), 1e-3, relative=True)
    args = [torch.from_numpy(x).cuda().repeat(n // 2, *[1] * (x.ndim - 1)) for x in (sums, G, C)]
    ws = torch.empty(cb.cb_ridge_solve_workspace_bytes(dx, dt, n), dtype=torch.uint8, device="cuda")
    maps = torch.full((n, dx + 1, dt), 7.0, device="cuda")
    info = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cb.cb_ridge_solve_centered_ws(*args, 1e-3, REL, maps, info, ws)
    assert (info.cpu().numpy() == 0).all() and (io == 0).all()
    for m in range(2):
        assert bool((maps[m::2] == maps[m]).all())
        assert _relF(maps[m].double().cpu().numpy(), W[m]) < 1e-6


# How long an fp32 sum runs: whole numbers whose sums are exact in fp32 over 16 tiles (below 2^24) but not over 64 (4e7).
# 512 items and 64 tiles are 4 chunks of 16 tiles, so only three additions of chunks round: by at most half of 2, 2 and 4.
def test_stats_sums_stay_short(cb):
    L, Ls, H, d, T = 64, 4, 8, 64, 2048
    rows = [(l, h, z, l % Ls, h, 0) for l in range(L) for z in range(2) for h in range(H)]
    names = ("tgt_layer", "tgt_head", "kv", "src_layer", "src_head", "weight_row")
    hm = {k: np.asarray(v, dtype=np.int32) for k, v in zip(names, zip(*rows))}
    g = torch.Generator(device="cuda").manual_seed(3)
    src = torch.randint(64, 201, (Ls, 2, 1, H, T, d), generator=g, device="cuda").bfloat16()
    tgt = torch.randint(64, 201, (L, 2, 1, H, T, d), generator=g, device="cuda").bfloat16()
    w = torch.ones((1, T), device="cuda")
    plan = cb.cb_plan_create(hm, src, tgt, T)
    G, C = torch.zeros((len(rows), d + 1, d + 1), device="cuda"), torch.zeros((len(rows), d + 1, d), device="cuda")
    cb.cb_stats_accumulate(plan, src, tgt, w, G, C)
    for m in range(0, len(rows), 37):
        l, h, z, s, _, _ = rows[m]
        x = torch.cat([src[s, z, 0, h].double(), torch.ones((T, 1), dtype=torch.float64, device="cuda")], dim=1)
        y = tgt[l, z, 0, h].double()
        assert 2 ** 25 < float((x.t() @ x)[0, 0]) < 2 ** 26
        assert float((G[m].double() - x.t() @ x).abs().max()) <= 4 and float((C[m].double() - x.t() @ y).abs().max()) <= 4


# Rotary statistics of plans with an item of a single map, whose other waves only copy and turn: chunks of several tiles,
# whole and ragged ones.  The products are bit for bit those of turned copies (the bias sums may round differently).
@pytest.mark.parametrize("maps", [1, 3])
@pytest.mark.parametrize("d,style,T", [(128, 0, 2048), (128, 1, 2090), (64, 0, 2090), (64, 1, 2048)])
def test_stats_rope_single_map_items(cb, d, style, T, maps):
    rows = [(0, 0, 0, 0, 0, 0), (1, 0, 1, 1, 0, 0), (2, 0, 0, 2, 0, 0)][:maps]
    names = ("tgt_layer", "tgt_head", "kv", "src_layer", "src_head", "weight_row")
    hm = {k: np.asarray(v, dtype=np.int32) for k, v in zip(names, zip(*rows))}
    g = torch.Generator(device="cuda").manual_seed(T + style)
    src = torch.randn((3, 2, 6, 1, T, d), generator=g, device="cuda").bfloat16()
    tgt = torch.randn((3, 2, 6, 1, T, d), generator=g, device="cuda").bfloat16()
    w = torch.rand((1, 6 * T), generator=g, device="cuda")
    tabs = [torch.empty((T + 7, d // 2, 2), device="cuda") for _ in range(2)]
    for t, theta in zip(tabs, (1e4, 1e6)):
        cb.cb_rope_table(theta, d, T + 7, t)
    plan = cb.cb_plan_create(hm, src, tgt, 6 * T)
    out = []
    for fused in (True, False):
        G, C = torch.zeros((maps, d + 1, d + 1), device="cuda"), torch.zeros((maps, d + 1, d), device="cuda")
        if fused:
            cb.cb_stats_accumulate_rope(plan, src, tgt, w, G, C, *(cb.rope_spec(t, style, 7) for t in tabs))
        else:
            turned = [x.clone() for x in (src, tgt)]
            for x, y, t in zip((src, tgt), turned, tabs):
                cb.cb_rope(x, y, t, style, True, 7)
            cb.cb_stats_accumulate(plan, *turned, w, G, C)
        out.append((G[:, :d, :d], C[:, :d]))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
