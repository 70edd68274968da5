"""Construction of the model matrix at the sizes where its work is split
differently: uniform edges, long rows."""
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


# two workgroups' pairs in the edges at up to 20 480 values each, atomics from
# one more on; 319 and 320 workgroups past that
@pytest.mark.parametrize("N,B", [(1, 1), (40960, 3), (40961, 3), (6_600_000, 638),
                                 (6_600_000, 639)])
def test_uniform_edges_bitexact(vup, orc, N, B):
    f = np.random.default_rng(N + B).normal(size=N)
    f[N // 2] = np.nan if N > 1 else 1.0
    f[-1] = 7.5  # the largest at the end
    assert np.array_equal(_cpu(vup.uniform_edges(torch.from_numpy(f).to(DEV), B)),
                          orc.uniform_edges(f, B))


@pytest.mark.parametrize("n", [(65536,), (3, 2048), (3, 2049), (2, 4127), (9000, 2051)])
def test_runs_of_long_rows_bitexact(vup, n):
    """Rows of one segment of 64 blocks of 32 cells, of just more, of two and a
    few cells, of 32; and more segments than one workgroup scans."""
    B, nL = 30, n[-1]
    rng = np.random.default_rng(nL)
    f = rng.integers(-1, B + 1, size=int(np.prod(n))).astype(np.float64)  # some outside
    f[rng.random(f.size) < 0.7] = 5.0
    g = vup.make_grid(n, (0.0,) * len(n), (1.0,) * len(n))
    e = torch.arange(0.0, B + 1, dtype=torch.float64, device=DEV) - 0.5
    mm = vup.build_model_matrix(g, torch.from_numpy(f).to(DEV), e)
    code = np.where((f >= 0) & (f < B), 4 * f, 4 * B).astype(np.int64).reshape(-1, nL)
    start = np.ones(code.shape, dtype=bool)
    start[:, 1:] = code[:, 1:] != code[:, :-1]
    count = start.sum(1)
    ptr = np.r_[0, np.cumsum(count + 1)]
    assert np.array_equal(_cpu(mm.rowptr), ptr)
    recs = np.full(ptr[-1], nL | (4 * B << 16), dtype=np.int64)  # the terminators
    r, c = np.nonzero(start)
    recs[np.arange(len(r)) + r] = c | (code[start] << 16)
    assert np.array_equal((_cpu(mm.runs).astype(np.int64) & 0xFFFFFFFF)[:len(recs)], recs)
    idx = (_cpu(mm.runidx).astype(np.int64) & 0xFFFF).reshape(-1, mm.mm.pitch)[:, :nL]
    assert np.array_equal(idx, np.cumsum(start, axis=1) - 1)
    assert int(mm._view(mm.mm.off_counters, torch.int64, 8)[4]) == count.sum()
