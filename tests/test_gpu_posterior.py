"""The posterior at the sizes where its kernels change: rows per workgroup, bins
per workgroup, factor tables."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module")
def vup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_11246_amd as v
    v.lib()
    return v


def _cpu(t):
    return t.detach().cpu().numpy()


# a row per workgroup, long and short; two rows for all but the last workgroup,
# and for all; four and a bit
@pytest.mark.parametrize("n,C,n_sel", [((1, 1024), 1, 3), ((16000,), 2, 2), ((7, 12), 1, 512),
                                       ((8, 12), 2, 512), ((300, 2052), 1, 29)])
def test_posterior_by_rows_per_workgroup(vup, n, C, n_sel):
    """post = sum_c w_c N_c(x) / Z_c / P[bin] cell by cell: FP32 factors of an
    ulp, their product and two roundings, so 16 units of 2^-24."""
    d, B = len(n), 30
    rng = np.random.default_rng(n[-1])
    g = vup.make_grid(n, (-1.0,) * d, (1.5,) * d)
    f = rng.normal(size=int(np.prod(n)))
    mm = vup.build_model_matrix(g, torch.from_numpy(f).to(DEV),
                                torch.linspace(-1.5, 1.5, B + 1, dtype=torch.float64, device=DEV))
    mu = rng.uniform(-1.0, 1.5, size=(n_sel, C, d))
    sg = rng.uniform(0.1, 0.5, size=(n_sel, C, d))
    w = rng.dirichlet(np.ones(C), size=n_sel)
    P, Z = vup.propagate(mm, mu, sg, w if C > 1 else None)
    post, _ = vup.posterior(mm, mu, sg, w if C > 1 else None, np.arange(n_sel), P, Z)
    post, P, Z, b = _cpu(post), _cpu(P).astype(np.float64), _cpu(Z), _cpu(mm.bin)
    win = _cpu(vup.windows(g, mu, sg, weight=w if C > 1 else None))
    for t in range(n_sel):
        want = 0.0
        for c in range(C):
            p = np.ones(())
            for i in range(d):
                x = -1.0 + (np.arange(n[i]) + 0.5) * (2.5 / n[i])
                q = np.exp(-0.5 * ((x - mu[t, c, i]) / sg[t, c, i]) ** 2)
                j = np.arange(n[i])
                q[(j < win[t, c, i, 0]) | (j > win[t, c, i, 1])] = 0.0
                p = np.multiply.outer(p, q)
            want = want + (w[t, c] if C > 1 else 1.0) / Z[t, c] * p.ravel()
        pb = np.where(b >= 0, P[t][np.maximum(b, 0)], 0.0)
        want = np.where(pb > 0, want / np.where(pb > 0, pb, 1.0), 0.0)
        assert np.all(np.abs(post[t] - want) <= 16 * 2.0 ** -24 * want), t


# from post (tables too long for few bins), from tables with four bins to a
# workgroup, five, and sixteen with a quarter of a wave each
@pytest.mark.parametrize("n,B,n_sel", [((8000,), 166, 1), ((8000,), 167, 1), ((60, 70), 31, 3),
                                       ((60, 70), 1031, 5), ((60, 70), 1638, 10),
                                       ((60, 70), 1639, 10)])
def test_means_by_bins_per_workgroup(vup, n, B, n_sel):
    """E[x | y in b] against the sums over the posterior of the same call: FP64,
    so within 2 (m + 8) 2^-53 of the sum of the m terms' magnitudes."""
    d = len(n)
    rng = np.random.default_rng(B)
    g = vup.make_grid(n, (-1.0,) * d, (1.5,) * d)
    f = torch.from_numpy(rng.normal(size=int(np.prod(n)))).to(DEV)
    mm = vup.build_model_matrix(g, f, vup.uniform_edges(f, B))
    mu = rng.uniform(-1.0, 1.5, size=(n_sel, 1, d))
    sg = rng.uniform(0.1, 0.5, size=(n_sel, 1, d))
    P, Z = vup.propagate(mm, mu, sg)
    post, mean = vup.posterior(mm, mu, sg, None, np.arange(n_sel), P, Z)
    post, mean, b = _cpu(post).astype(np.float64), _cpu(mean), _cpu(mm.bin)
    x = np.meshgrid(*[-1.0 + (np.arange(m) + 0.5) * (2.5 / m) for m in n], indexing="ij")
    count = np.bincount(b, minlength=B)
    for t in range(n_sel):
        for i in range(d):
            want = np.bincount(b, weights=post[t] * x[i].ravel(), minlength=B)
            size = np.bincount(b, weights=post[t] * 2.5, minlength=B)
            assert (np.abs(mean[t, :, i] - want) <= 2 * (count + 8) * 2.0 ** -53 * size).all(), t
