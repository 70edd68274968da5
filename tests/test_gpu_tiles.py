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


# A column factor is a whole number of units of 2^-25 of the tile's largest
# factor or finer, so within 4 deviations (factors above e^-8) it is off by at
# most e^8 2^-26 = 4.4e-5 of itself; row factors are FP64; a bin's entry is
# rounded to 2^-51 of a bound of the pdf's mass (at most about 8 times the mass,
# for a mean in a corner of the grid), and a bin has some hundreds of entries in
# these windows: 1e-12 of the mass. The output is FP32.
REL, ABS = np.exp(8.0) * 2.0 ** -26 + 2.0 ** -24, 1e-12


@pytest.mark.parametrize("n,B,cells", [((256, 256), 64, (1.0, 30.0)), ((300, 200), 40, (0.5, 4.0)),
                                       ((512, 512), 128, (8.0, 60.0))])
def test_small_bins_keep_their_digits(vup, orc, n, B, cells):
    """Every bin by its mass, the posterior's sum over the cells of a bin, and
    the normalisers, on maps of 16 384 pdfs."""
    K, m = 16384, 160
    mm, b = _matrix(vup, orc, n, B)
    mu, sg = _gaussians(n, LO, HI, K, cells, B)
    P, Z = vup.propagate(mm, mu, sg)
    at = np.random.default_rng(1).choice(K, size=m, replace=False)
    p = _cpu(P)[at].astype(np.float64)
    po, zo = orc.propagate(n, LO, HI, b, B, mu[at], sg[at])
    has = po > 0
    err = np.abs(p - po)[has] / po[has]
    _say(f"[small bins {n} B={B} {cells}] smallest {po[has].min():.1e}, largest error over the "
         f"bar {(err / (REL + ABS / po[has])).max():.2f}")
    assert (po[has] < 1e-7).any()
    assert (err <= REL + ABS / po[has]).all()
    np.testing.assert_allclose(_cpu(Z)[at], zo, rtol=1e-7)
    post, _ = vup.posterior(mm, mu, sg, None, at, P, Z)
    post = _cpu(post).astype(np.float64)
    for t in range(m):
        s = np.bincount(b, weights=post[t], minlength=B)[has[t]]
        # (its factors are FP32: a few units of 2^-24)
        assert (np.abs(s - 1.0) <= 2 * (REL + ABS / po[t][has[t]]) + 2.0 ** -20).all(), t


def test_narrow_pdfs(vup, orc):
    """Deviations far below a cell, next to wide ones and outside the grid."""
    n, B, K = (131, 200), 40, 16384
    mm, b = _matrix(vup, orc, n, B)
    rng = np.random.default_rng(6)
    h = np.array([6.0 / 131, 6.0 / 200])
    mu = rng.uniform(-3 - 3 * h, 3 + 3 * h, size=(K, 1, 2))
    sg = 10.0 ** rng.uniform(-4, 1, size=(K, 1, 2)) * h
    sg[:2000] = 10.0 ** rng.uniform(-12, -4, size=(2000, 1, 2)) * h
    P, Z = vup.propagate(mm, mu, sg, n_sigma=6.0)
    P, Z = _cpu(P).astype(np.float64), _cpu(Z)[:, 0]
    Po, Zo = orc.propagate(n, LO, HI, b, B, mu, sg, n_sigma=6.0)
    Zo = Zo[:, 0]
    # densities below FP64's range have no P: vup_propagate's rows, bit for bit
    # (none at the end of the range are compared)
    ok = (Zo > 1e-290) | (Po == 0).all(1)
    none = np.nonzero((Zo == 0) & ~ok)[0][:8000]
    assert ok.sum() > 3000 and len(none) > 3000
    Pn, _ = vup.propagate(mm, mu[none], sg[none], n_sigma=6.0)
    assert np.array_equal(P[none], _cpu(Pn), equal_nan=True) and np.isnan(P[none]).any()
    assert np.isfinite(P[ok]).all() and np.abs(P - Po)[ok].sum(1).max() <= 2e-5
    np.testing.assert_allclose(Z[ok], Zo[ok], rtol=2e-6)
    w = _cpu(vup.windows(mm.grid, mu, sg, n_sigma=6.0))[:, 0]
    one = (w[..., 0] == w[..., 1]).all(1) & ok & (Zo > 0)  # a single cell
    assert one.sum() > 50 and (P[one].max(1) == 1.0).all() and (P[one].sum(1) == 1.0).all()


def test_workspace_sets_the_passes(vup, orc):
    """Any workspace between the least and the full one gives the same results:
    the pdfs are taken in passes, and by vup_propagate's kernel when a pass
    would be too small."""
    n, B, K = (190, 150), 300, 70001
    mm, _ = _matrix(vup, orc, n, B)
    mu, sg = _gaussians(n, LO, HI, K, (0.5, 20.0), 9)
    sg[17] = -1.0
    mu, sg = torch.from_numpy(mu).to(DEV), torch.from_numpy(sg).to(DEV)
    d, lib = vup._dists(mu, sg, None, 4.0), vup.lib()
    m, dd = ctypes.byref(mm.mm), ctypes.byref(d)
    least = lib.vup_propagate_tiled_workspace_bytes(m, dd, 0)
    full = lib.vup_propagate_tiled_full_workspace_bytes(m, dd, 0)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def call(nb):
        ws = torch.full((nb,), 0xA5, dtype=torch.uint8, device=DEV)
        P = torch.full((K, B), -7.0, device=DEV)
        Z = torch.full((K, 1), -7.0, dtype=torch.float64, device=DEV)
        assert lib.vup_propagate_tiled(m, dd, 0, ptr(ws), nb, ptr(P), ptr(Z), stream) == 0
        return P.nan_to_num(-1.0), Z.nan_to_num(-1.0)

    ref = call(full)
    assert least < full
    for share in (2, 4):  # (three and four passes: the least part does not shrink with K)
        P, Z = call(least + (full - least) // share)
        assert torch.equal(P, ref[0]) and torch.equal(Z, ref[1]), share
    P, Z = call(least)
    Pp, Zp = vup.propagate(mm, mu[:5000], sg[:5000])  # the per-pdf kernel
    assert torch.equal(P[:5000], Pp.nan_to_num(-1.0)) and torch.equal(Z[:5000], Zp.nan_to_num(-1.0))
    assert (P - ref[0]).abs().sum(1).max() <= 4e-5


def test_tiles_of_several_passes(vup, orc):
    """Tiles whose bins need up to three passes, with cells without a bin among
    them, next to tiles of one; and the count of passes that decides on the tiles."""
    n, K, m = (1408, 256), 16384, 160
    rows = np.r_[np.full(128, 2.3), np.full(n[0] - 128, 0.25)].cumsum()
    f = (rows[:, None] + 0.2 * np.arange(n[1])[None, :]).ravel()
    f[::977] = np.nan
    e = np.arange(40.0, np.nanmax(f) + 1.0)  # the first 40 bins' cells have none
    B = len(e) - 1
    b = orc.bins(f, e)
    g = vup.make_grid(n, LO, HI)
    mm = vup.build_model_matrix(g, torch.from_numpy(f).to(DEV), torch.from_numpy(e).to(DEV))
    passes = 0
    for y in range(0, n[0], 128):
        for x in range(0, n[1], 64):
            q = b.reshape(n)[y:y + 128, x:x + 64]
            q = q[q >= 0]
            passes += (q.max() - q.min()) // 120 + 1
    tiles = (n[0] // 128) * (n[1] // 64)
    # (the counter holds those past the first over each tile)
    assert int(mm._view(mm.mm.off_counters, torch.int64, 8)[5]) == passes - tiles > 0
    assert mm.sweep == "runs" and mm.mm.reserved == 1  # the tiles pay
    mu, sg = _gaussians(n, LO, HI, K, (1.0, 40.0), 11)
    mu[:K // 2, 0, 0] = np.random.default_rng(2).uniform(-3.0, -2.4, size=K // 2)  # the steep rows
    P, Z = vup.propagate(mm, mu, sg)
    P, reached = _cpu(P), _reached(vup, mm, b, mu, sg, B)
    assert (P[~reached] == 0).all()
    at = np.random.default_rng(3).choice(K // 2, size=m, replace=False)
    po, zo = orc.propagate(n, LO, HI, b, B, mu[at], sg[at])
    p, has = P[at].astype(np.float64), po > 0
    err = np.abs(p - po)[has] / po[has]
    _say(f"[several passes] {passes} of {tiles} tiles, largest error over the bar "
         f"{(err / (REL + ABS / po[has])).max():.2f}")
    assert (err <= REL + ABS / po[has]).all()
    np.testing.assert_allclose(_cpu(Z)[at], zo, rtol=1e-7)
    # too many passes: found not to pay
    f = np.add.outer(2.3 * np.arange(256.0), 0.2 * np.arange(256.0)).ravel()
    mm = vup.build_model_matrix(vup.make_grid((256, 256), LO, HI), torch.from_numpy(f).to(DEV),
                                torch.arange(0.0, f.max() + 1.0, dtype=torch.float64, device=DEV))
    assert mm.sweep == "runs" and mm.mm.reserved == 2


def test_without_memory_for_the_workspace(vup, orc, monkeypatch):
    """A call that finds no memory for the tiles' workspace is the per-pdf form's."""
    mm, _ = _matrix(vup, orc, (190, 150), 20)
    mu, sg = _gaussians((190, 150), LO, HI, 16384, (0.5, 20.0), 3)
    ref = vup.propagate(mm, mu, sg)
    empty = torch.empty

    def no_bytes(*a, **kw):
        if kw.get("dtype") is torch.uint8:
            raise torch.OutOfMemoryError("none left")
        return empty(*a, **kw)

    monkeypatch.setattr(vup.torch, "empty", no_bytes)
    P, Z = vup.propagate(mm, mu, sg)
    monkeypatch.undo()
    part = vup.propagate(mm, mu[:5000], sg[:5000])
    assert torch.equal(P[:5000], part[0]) and torch.equal(Z[:5000], part[1])
    assert (P - ref[0]).abs().sum(1).max() <= 4e-5


def test_tiled_graph_capture(vup, orc):
    """A captured tiled propagation, replayed over new pdfs with eager calls in
    between, gives the eager results."""
    n, B, K = (256, 256), 64, 16384
    mm, _ = _matrix(vup, orc, n, B)
    sets = [[torch.from_numpy(a).to(DEV) for a in _gaussians(n, LO, HI, K, (0.3, 30.0), s)]
            for s in range(3)]
    sets[1][1][100:200] = -1.0  # invalid ones among them
    mu, sg = sets[0][0].clone(), sets[0][1].clone()
    vup.propagate(mm, mu, sg)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P, Z = vup.propagate(mm, mu, sg)
    for i in (0, 1, 2, 1, 0):
        mu.copy_(sets[i][0])
        sg.copy_(sets[i][1])
        ref = vup.propagate(mm, sets[i][0], sets[i][1])
        graph.replay()
        torch.cuda.synchronize()
        for a, r in zip((P, Z), ref):
            assert torch.equal(a.nan_to_num(-1.0), r.nan_to_num(-1.0)), i
