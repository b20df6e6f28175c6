"""The anti-trapping current leaves out faces where no lane has a solid-liquid
interface: grids that are mostly exact bulk (waves that skip beside waves that do
not, an interface across a strip's edge and across a row segment), and one value
that is not finite in the bulk, which has to spread as the oracle spreads it.
Against the oracle, four steps: FP64 rounding stays below 1e-12."""
import numpy as np
import pytest

from test_gpu_antitrapping import oracle_run_at, run_gpu_at
from test_gpu_parity import variant

pytestmark = pytest.mark.gpu


def bulk_case(n, bc, N, K, dim, ext):
    """Liquid everywhere but a blob of solid on cell 60 of x (a strip's edge), with an interface of a few cells."""
    p = variant(dim=dim, N=N, K=K, n=n, bc=bc, seed=11, potential="obstacle" if ext == "obstacle" else "well")
    if ext == "slopes":
        p.Bt[:N, :K - 1] = 0.05
    rng = np.random.default_rng(4)
    shape = tuple(reversed(n[:dim]))
    ax = [np.arange(s) - c for s, c in zip(shape, [min(s // 2, 14) for s in shape[:-1]] + [60])]
    r = np.sqrt(sum(g.astype(float) ** 2 for g in np.meshgrid(*ax, indexing="ij")))
    solid = np.clip((6.0 - r) / 8.0 + 0.5, 0.0, 1.0)  # exact 0 and 1 outside the interface
    phi = np.zeros((N,) + shape)
    share = rng.dirichlet(np.ones(N - 1), size=shape) if N > 2 else np.ones(shape + (1,))
    for a in range(N - 1):
        phi[a] = solid * share[..., a]
    phi[N - 1] = 1.0 - phi[:N - 1].sum(axis=0)
    mu = rng.uniform(-0.05, 0.05, size=(K - 1,) + shape)
    return p, phi, mu


@pytest.mark.parametrize("n,bc,N,K,ext", [
    ((190, 40, 1), (0, 0, 0), 3, 3, None), ((190, 40, 1), (1, 1, 0), 2, 2, "slopes"),
    ((131, 33, 1), (0, 1, 0), 3, 2, "obstacle"), ((130, 12, 14), (0, 1, 0), 2, 2, None),
    ((126, 9, 11), (1, 0, 1), 3, 3, "slopes"),
])
@pytest.mark.parametrize("fault", [None, np.nan, np.inf])
def test_bulk_faces_against_the_oracle(n, bc, N, K, ext, fault):
    dim = 3 if n[2] > 1 else 2
    p, phi, mu = bulk_case(n, bc, N, K, dim, ext)
    steps = 4
    if fault is not None:
        mu[(0,) + (4,) * (dim - 1) + (110,)] = fault  # in the melt, away from the blob
        steps = 1
    print(f"bulk {n[:dim]} N={N} K={K} {ext} fault {fault}", flush=True)
    with np.errstate(all="ignore"):
        want = oracle_run_at(phi, mu, 5, steps, p)
    got = run_gpu_at(p, phi, mu, steps, step0=5)
    bad = ~np.isfinite(want[1])
    assert np.array_equal(~np.isfinite(got[1]), bad) and bad.any() == (fault is not None)
    assert np.max(np.abs(got[1] - want[1])[~bad]) <= 1e-12
    ok = ~bad.any(axis=0) & np.isfinite(want[0]).all(axis=0)
    assert np.max(np.abs(got[0] - want[0])[:, ok]) <= 1e-12
