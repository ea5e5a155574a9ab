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
