"""Every tile of the dense product at ragged sizes: each case states the tile that
its sizes must be given (cts_layer_plan), so that another choice shows here, and
is compared row by row with a float64 evaluation on the tokens at the edges of
the sorted order's tiles and runs and on random ones; every output element is
written."""
import numpy as np
import pytest
import torch

import paper_2407_00066_amd as cts

from _gpu_helpers import TOL, host, row_rel_err, say

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32


class Layer:
    """Operands of one layer on the GPU (d_outs: the modules of one input)."""

    def __init__(self, seed, T, d_in, d_outs, r, n, K, ids, dtype=BF16):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        rs = np.random.default_rng(seed)
        if ids == "prompts":
            aid = np.repeat(rs.integers(0, n, T), rs.integers(16, 200, T))[:T]
        elif ids == "once":                       # one adapter takes the batch, every other one token
            aid = rs.permutation(np.concatenate([np.arange(n), np.full(T - n, n // 2)]))
        else:
            aid = rs.integers(0, n, T) if ids == "uniform" else np.minimum(rs.zipf(1.3, T) - 1, n - 1)
        self.T, self.r, self.n, self.K, self.dtype, self.d_in, self.d_outs = T, r, n, K, dtype, d_in, list(d_outs)
        self.aid = torch.from_numpy(aid.astype(np.int32)).cuda()
        self.cof = torch.from_numpy(rs.permutation(np.arange(n) % K).astype(np.int32)).cuda()
        M = len(d_outs)
        self.x = self.draw((T, d_in), 1.0)
        self.W = [self.draw((d, d_in), 1.0 / d_in) for d in d_outs]
        self.U = [self.draw((K, d, r), 1.0 / r) for d in d_outs]
        self.Vt = self.draw((K, M * r, d_in), 1.0 / d_in)
        self.S = [self.draw((n, r, r), 1.0 / r) for _ in d_outs]

    def draw(self, shape, var):
        return (torch.randn(shape, generator=self.g, device="cuda") * var ** 0.5).to(self.dtype)

    def plan(self, multi=False):
        p = cts.make_problem(self.T, self.d_in, self.d_outs[0], r=self.r, n_adapters=self.n, n_clusters=self.K,
                             dtype=cts.CTS_BF16 if self.dtype == BF16 else cts.CTS_F32)
        return cts.layer_plan(p, d_outs=self.d_outs if multi else None)

    def sample(self):
        """Tokens at both sides of every 64-position edge near the ends and of
        some runs' edges, and random ones."""
        perm, offs = cts.sort_by_cluster(self.aid, self.cof, self.n, self.K)
        perm, offs = perm.cpu().numpy(), offs.cpu().numpy()
        at = {0, 1, 15, 16, 63, 64, 127, 128, 255, 256, 257, self.T - 2, self.T - 1, self.T // 256 * 256}
        at |= {int(o) + s for o in offs[:40] for s in (-1, 0)}
        at |= set(np.random.default_rng(3).integers(0, self.T, 60).tolist())
        return torch.from_numpy(perm[sorted(a for a in at if 0 <= a < self.T)].astype(np.int64)).cuda()

    def expected(self, m, rows, ranks=None):
        r, seg = self.r, self.cof.long()[self.aid[rows].long()]
        x = self.x[rows].double()
        y = x @ self.W[m].double().t()
        for q in range(rows.numel()):
            k = int(seg[q])
            rk = r if ranks is None else int(ranks[k])
            z = self.Vt[k, m * r:m * r + rk].double() @ x[q]
            y[q] += self.U[m][k, :, :rk].double() @ (self.S[m][int(self.aid[rows[q]])][:rk, :rk].double() @ z)
        return y


def _same(y, want, rows, dtype=BF16):
    assert bool(torch.isfinite(y.float()).all())              # (every element written: y began as NaN)
    assert row_rel_err(host(y[rows]), want.cpu().numpy()) <= TOL["bf16" if dtype == BF16 else "f32"]


@pytest.mark.parametrize("T,d_in,d_out,r,n,K,ids", [
    (2777, 3000, 5000, 48, 500, 16, "prompts"),   # every side ragged; a rank of one and a half units
    (2300, 2056, 5000, 128, 90, 3, "prompts"),    # 65 dense units (the last of 8), four units a run, few runs
    (2300, 2056, 5000, 128, 900, 60, "uniform"),  # as many runs as fit: the units that skip columns
    (2304, 3008, 5000, 64, 900, 60, "uniform"),   # aligned rows, whole units, many runs
    (2305, 3008, 5000, 24, 90, 3, "prompts"),     # a column tile of one token
    (4096, 128, 8192, 64, 200, 20, "uniform"),    # exactly four dense units: no whole round of the ring
    (4090, 136, 16136, 40, 200, 8, "uniform"),    # five, the last of 8; a row tile of 8 rows
    (4090, 152, 14344, 8, 20, 1, "prompts"),      # one run of one unit over every tile
    (4096, 288, 16392, 16, 400, 70, "uniform"),   # nine dense units, some five runs of one unit a tile
])
def test_prefill_tile(T, d_in, d_out, r, n, K, ids):
    w = Layer(7000 + T + d_in + r, T, d_in, [d_out], r, n, K, ids)
    assert w.plan() == (256, 256, 1, "fused")
    rows = w.sample()
    say("prefill tile T=%d %dx%d r=%d K=%d" % (T, d_in, d_out, r, K))
    want = w.expected(0, rows)
    for dt in (BF16, F32):
        out = torch.full((T, d_out), float("nan"), dtype=dt, device="cuda")
        _same(cts.apply(w.x, w.aid, w.cof, w.W[0], w.U[0], w.Vt, w.S[0], out=out), want, rows)
    ranks = np.random.default_rng(5).integers(0, r // 8 + 1, K) * 8
    out = torch.full((T, d_out), float("nan"), dtype=BF16, device="cuda")
    rk = torch.from_numpy(ranks.astype(np.int32)).cuda()
    _same(cts.apply_ranked(w.x, w.aid, w.cof, w.W[0], w.U[0], w.Vt, w.S[0], rk, out=out), w.expected(0, rows, ranks), rows)


def test_prefill_tile_needs_four_units():
    """One feature block short of the four units that the 256 x 256 tile's setup
    loads whole, another tile is taken."""
    for d_in, tile in ((120, (256, 128)), (128, (256, 256))):
        p = cts.make_problem(4096, d_in, 8192, r=64, n_adapters=200, n_clusters=20)
        assert cts.layer_plan(p)[:2] == tile


@pytest.mark.parametrize("T,d_in,d_outs,r,n,K,ids,plan", [
    (512, 4096, (14336, 14088), 16, 40, 4, "uniform", (256, 256, 1, "grouped")),
    (512, 1032, (14088, 14336, 8), 64, 400, 50, "uniform", None),
    (300, 1032, (520, 264, 8), 48, 50, 5, "zipf", None),
    (40, 264, (16392, 520), 40, 20, 4, "uniform", (64, 64, 1, "fused")),      # 266 row tiles: a launch each
    (64, 2056, (16384, 520), 128, 20, 9, "uniform", (64, 64, 1, "fused")),    # the narrow module in four pieces
    (17, 4104, (8200, 8200), 8, 5, 2, "uniform", (64, 64, 1, "fused")),       # 258 row tiles
])
def test_modules(T, d_in, d_outs, r, n, K, ids, plan):
    """Modules of unequal widths in one call, grouped in one launch or not."""
    w = Layer(7500 + T + d_in, T, d_in, d_outs, r, n, K, ids)
    assert plan is None or w.plan(multi=True) == plan
    rows = w.sample()
    say("modules T=%d %d -> %s r=%d K=%d: %s" % (T, d_in, d_outs, r, K, w.plan(multi=True)))
    ys = cts.apply_multi(w.x, w.aid, w.cof, w.W, w.U, w.Vt, w.S,
                         outs=[torch.full((T, d), float("nan"), dtype=BF16, device="cuda") for d in d_outs])
    for m, y in enumerate(ys):
        want = w.expected(m, rows)
        # (a module of 8 outputs has no large one in every row to measure by)
        scale = w.expected(0, rows).abs().amax(1, keepdim=True)
        assert bool(torch.isfinite(y.float()).all())
        assert float(((y[rows].double() - want).abs() / scale).max()) <= TOL["bf16"], m


@pytest.mark.parametrize("T,d_in,d_out,r,tile", [
    (4096, 288, 16392, 16, (256, 256)),
    (2048, 256, 8192, 64, (256, 128)),
    (700, 264, 5000, 40, (128, 128)),
])
def test_adapter_term_of_many_runs(T, d_in, d_out, r, tile):
    """More than 64 cluster runs in one tile's tokens (a tile lists them 64 at a
    time), with W = 0: the error is then measured by the adapter term alone."""
    n = 150
    w = Layer(7900 + T, T, d_in, [d_out], r, n, n, "once")
    w.W[0].zero_()
    assert w.plan()[:2] == tile
    seg = np.sort(w.cof.cpu().numpy()[w.aid.cpu().numpy()])
    assert max(len(set(seg[i:i + tile[1]])) for i in range(0, T, tile[1])) > 64
    rows = w.sample()
    say("many runs T=%d %dx%d r=%d" % (T, d_in, d_out, r))
    args = (w.x, w.aid, w.cof, w.W[0], w.U[0], w.Vt, w.S[0])
    out = torch.full((T, d_out), float("nan"), dtype=BF16, device="cuda")
    _same(cts.apply(*args, out=out), w.expected(0, rows), rows)
    ranks = np.arange(n) % (r // 8) * 8 + 8
    rk = torch.from_numpy(ranks.astype(np.int32)).cuda()
    _same(cts.apply_ranked(*args, rk), w.expected(0, rows, ranks), rows)


@pytest.mark.parametrize("T,d_in,d_out,r,K", [
    (1, 8, 16392, 8, 1),          # one token, one k-tile of 8
    (40, 264, 16400, 128, 9),     # three dense k-tiles, the last of 8: the prologue takes adapter k-tiles
    (64, 1032, 16648, 72, 30),    # a last row tile of 8 rows
])
def test_wide_decode_tile(T, d_in, d_out, r, K):
    """More than 256 row tiles: the 64 x 64 tile that adds U_k Z' itself."""
    w = Layer(7800 + T, T, d_in, [d_out], min(r, d_in), 40, K, "uniform")
    assert w.plan() == (64, 64, 1, "fused")
    rows = w.sample()
    say("wide decode T=%d %dx%d r=%d" % (T, d_in, d_out, r))
    args = (w.x, w.aid, w.cof, w.W[0], w.U[0], w.Vt, w.S[0])
    for dt in (BF16, F32):
        out = torch.full((T, d_out), float("nan"), dtype=dt, device="cuda")
        _same(cts.apply(*args, out=out), w.expected(0, rows), rows)
    ranks = np.arange(K) % (w.r // 8 + 1) * 8
    rk = torch.from_numpy(ranks.astype(np.int32)).cuda()
    _same(cts.apply_ranked(*args, rk), w.expected(0, rows, ranks), rows)
