"""The tiled propagation's parts on the GPU: the entry lists that vup_bin builds
and what the sums over the tiles keep, against plain NumPy and the FP64 oracle."""
import ctypes
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"
LO, HI = (-3.0, -3.0), (3.0, 3.0)
NONE = 0xFFFF  # bin of an entry of cells without a bin


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def vup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_11246_amd as v
    v.lib()
    return v


def _cpu(t):
    return t.detach().cpu().numpy()


def _matrix(vup, orc, n, B, model="sincos2", share=1.0, lo=LO, hi=HI):
    """Model matrix in the run form over bins of `share` of the values' range,
    and the oracle's bins."""
    f = orc.eval_grid(n, lo, hi, model)
    e = orc.uniform_edges(f, B)
    if share != 1.0:
        c, r = 0.5 * (f.min() + f.max()), 0.5 * (f.max() - f.min()) * share
        e = np.linspace(c - r, c + r, B + 1)
    g = vup.make_grid(n, lo, hi)
    mm = vup.build_model_matrix(g, torch.from_numpy(f).to(DEV), torch.from_numpy(e).to(DEV),
                                resolve_sweep=False)
    mm.set_sweep_mode("runs")
    return mm, orc.bins(f, e)


# ---------------------------------------------------------------------------
# entry lists
# ---------------------------------------------------------------------------
def _lists(mm):
    """The chunks' lists, from the last sections of the model matrix's workspace:
    per block of 64 x 64 cells and chunk of four rows, (columns [n][4], bins [n])."""
    n0, n1 = mm.grid.n[0], mm.grid.n[1]
    nb = ((n0 + 63) // 64) * ((n1 + 63) // 64)
    up = lambda b: (b + 255) // 256 * 256
    blocks = int(mm.mm.ws_bytes) - up(nb * 16)
    chunks = blocks - up(nb * 16 * 16)
    cap = n0 * n1 // 10 + 64
    ent = _cpu(mm._view(chunks - up(cap * 8), torch.int32, 2 * cap)).astype(np.int64) & 0xFFFFFFFF
    ch = _cpu(mm._view(chunks, torch.int32, nb * 16 * 4)).reshape(nb * 16, 4)
    out = []
    for first, n in ch[:, :2]:
        e = ent.reshape(-1, 2)[first:first + n]
        out.append((np.stack([(e[:, 0] >> (8 * i)) & 255 for i in range(4)], 1), e[:, 1] & 0xFFFF))
    return out


def _rule(rows, w, none):
    """One rule's list over up to four rows of bin codes."""
    ends = [np.r_[np.nonzero(np.diff(r))[0] + 1, len(r)] for r in rows]
    at, col = [0] * len(rows), [0] * 4
    cols, bins = [], []
    while True:
        live = [i for i in range(len(rows)) if at[i] < len(ends[i])]
        if not live:
            return cols, bins
        code = {i: int(rows[i][col[i]]) for i in live}
        b = (min(code.values()) if w == 0 else max(code.values()) if w == 1 else
             min((col[i], code[i]) for i in live)[1])
        for i in live:
            if code[i] == b:
                col[i] = int(ends[i][at[i]])
                at[i] += 1
        cols.append(list(col))
        bins.append(NONE if b == none else b // 4)


def _reference_lists(b, n, B):
    """Shortest list of each chunk, of equally short ones the first rule's, made
    even by an entry that adds nothing; and how many chunks a rule that is one
    entry longer than an odd shortest list could have won after that."""
    code = np.where(b >= 0, 4 * b, 4 * B).reshape(n)
    out, close = [], 0
    for y in range(0, n[0], 64):
        for x in range(0, n[1], 64):
            blk = code[y:y + 64, x:x + 64]
            for r in range(0, 64, 4):
                rows = blk[r:r + 4]
                ls = [_rule(rows, w, 4 * B) for w in range(3)] if len(rows) else [([], [])]
                length = [len(l[0]) for l in ls]
                best = length.index(min(length))
                cols, bins = ls[best]
                close += len(cols) % 2 == 1 and any(m == len(cols) + 1 for m in length[:best])
                if len(cols) % 2:
                    cols, bins = cols + [cols[-1]], bins + [NONE]
                out.append((np.array(cols).reshape(-1, 4), np.array(bins)))
    return out, close


@pytest.mark.parametrize("n,B,share", [((256, 256), 64, 1.0), ((131, 200), 40, 0.6),
                                       ((512, 512), 128, 1.0)])
def test_entry_lists_do_not_depend_on_wave_order(vup, orc, n, B, share):
    mm, b = _matrix(vup, orc, n, B, share=share)
    ref, close = _reference_lists(b, n, B)
    _say(f"[entry lists {n} B={B}] {len(ref)} chunks, {close} with a rule one entry longer")
    assert close > 0
    for i, ((gc, gb), (rc, rb)) in enumerate(zip(_lists(mm), ref)):
        assert len(gb) == len(rb), i
        assert np.array_equal(gc, rc) and np.array_equal(gb, rb), i


def test_tiled_result_does_not_depend_on_the_build(vup, orc):
    """The same model matrix built again gives the same P, bit for bit."""
    n, B, K = (256, 256), 64, 16384
    rng = np.random.default_rng(3)
    mu = torch.from_numpy(rng.uniform(-3, 3, size=(K, 1, 2))).to(DEV)
    sg = torch.from_numpy(rng.uniform(0.05, 0.4, size=(K, 1, 2))).to(DEV)
    first = None
    for i in range(6):
        mm, _ = _matrix(vup, orc, n, B)
        P, Z = vup.propagate(mm, mu, sg)
        if first is None:
            first = P, Z
        assert torch.equal(P, first[0]) and torch.equal(Z, first[1]), i


# ---------------------------------------------------------------------------
# what the sums keep
# ---------------------------------------------------------------------------
def _gaussians(n, lo, hi, K, cells, seed):
    rng = np.random.default_rng(seed)
    h = (np.asarray(hi) - np.asarray(lo)) / np.asarray(n)
    mu = rng.uniform(lo, hi, size=(K, 1, 2))
    return mu, np.exp(rng.uniform(*np.log(cells), size=(K, 1, 2))) * h


def _reached(vup, mm, b, mu, sg, B):
    """[K][B]: the pdf's window has a cell of the bin (2-D prefix sums per bin)."""
    n = (mm.grid.n[0], mm.grid.n[1])
    w = _cpu(vup.windows(mm.grid, mu, sg))[:, 0].astype(np.int64)
    out = np.zeros((len(w), B), dtype=bool)
    b2 = b.reshape(n)
    for q in range(B):
        c = np.zeros((n[0] + 1, n[1] + 1), dtype=np.int64)
        c[1:, 1:] = (b2 == q).cumsum(0).cumsum(1)
        (l0, h0), (l1, h1) = (w[:, 0, 0], w[:, 0, 1] + 1), (w[:, 1, 0], w[:, 1, 1] + 1)
        out[:, q] = c[h0, h1] - c[l0, h1] - c[h0, l1] + c[l0, l1] > 0
    return out


@pytest.mark.parametrize("cells", [(0.5, 1.0), (1.0, 4.0), (4.0, 40.0)])
@pytest.mark.parametrize("n,B,share", [((256, 256), 64, 1.0), ((190, 150), 20, 0.6)])
def test_bins_outside_the_window_are_exact_zeros(vup, orc, n, B, share, cells):
    mm, b = _matrix(vup, orc, n, B, share=share)
    mu, sg = _gaussians(n, LO, HI, 16384, cells, B)
    P, _ = vup.propagate(mm, mu, sg)
    P, reached = _cpu(P), _reached(vup, mm, b, mu, sg, B)
    _say(f"[zeros {n} B={B} {cells}] {(~reached).sum()} bins out of reach, "
         f"{(P[~reached] != 0).sum()} of them with mass")
    assert (~reached).any() and (P[~reached] == 0).all()


def test_very_wide_pdfs(vup, orc):
    """Deviations up to the largest double: flat over the grid, Z the number of
    cells, P the share of each bin."""
    n, B, K = (131, 200), 40, 16384
    mm, b = _matrix(vup, orc, n, B)
    rng = np.random.default_rng(5)
    mu = rng.uniform(-3, 3, size=(K, 1, 2))
    sg = 10.0 ** rng.uniform(8, 308, size=(K, 1, 2))
    sg[:8, 0] = [[1e20, 1e20], [1e39, 1.0], [1.0, 1e45], [1e50, 1e50], [1e150, 1e300], [1e307, 1e307],
                 [1.7e308, 1.7e308], [2.0, 1e307]]
    P, Z = vup.propagate(mm, mu, sg)
    P, Z = _cpu(P).astype(np.float64), _cpu(Z)[:, 0]
    Po, Zo = orc.propagate(n, LO, HI, b, B, mu, sg)
    # FP32 output of sums with far more bits: the bar of the FP32 columns
    assert np.isfinite(P).all() and np.abs(P - Po).sum(1).max() <= 2e-5
    np.testing.assert_allclose(Z, Zo[:, 0], rtol=2e-6)
