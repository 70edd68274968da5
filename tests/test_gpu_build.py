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
