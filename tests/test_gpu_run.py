"""The evaluation kernel at the sizes where its cut of the work can go wrong:
sub-tiles, windows and staged pieces that end just before, at and past a
boundary, every stack class, datasets so wide or long that a tile is staged in
pieces, more programs than one workgroup lists; and the handlers' fast ranges,
at the bounds where they hand over to the general form.

Tolerances: outputs of additions and quotients are correctly rounded, so they
equal NumPy's float32 bit for bit; a reward is an integer.  A mean square has
a rounding of the residual (2^-24, twice in the square), of the square and of
a compensated sum (2^-23): below 2^-21.  Correlation scores take the oracle
gate's 1e-4."""
import numpy as np
import pytest

import oracle
from paper_2607_06731_amd import synth

pytestmark = pytest.mark.gpu


def _gp():
    import paper_2607_06731_amd as gp
    return gp


DEPTHS = (1, 2, 8, 9, 16, 17, 32)


def _sums(n_vars, copies):
    """Programs that push `depth` variables and add them up from the top."""
    progs, use = [], []
    for r in range(copies):
        for d in DEPTHS:
            v = [(r + 3 * k) % n_vars for k in range(d)]
            progs.append([synth.LOAD | (k << 8) for k in v] + [synth.ADD] * (d - 1))
            use.append(v)
    nodes = np.concatenate([np.array(p, np.uint32) for p in progs])
    offsets = np.concatenate([[0], np.cumsum([len(p) for p in progs])]).astype(np.int64)
    return nodes, offsets, use


@pytest.mark.parametrize("n_cases,n_vars,copies", [
    (1, 1, 1), (63, 2, 3), (128, 3, 1), (255, 2, 9), (256, 2, 40), (257, 5, 9), (511, 3, 9),
    (513, 11, 9), (1537, 3, 30), (3073, 5, 9), (4099, 1, 9), (40961, 3, 9), (100003, 7, 3),
    (700, 60, 5), (20000, 60, 3), (300, 127, 2), (300, 128, 3), (2100, 156, 2)])
def test_sums_over_all_classes(n_cases, n_vars, copies):
    gp = _gp()
    rng = np.random.default_rng(n_cases + n_vars)
    X = rng.uniform(-3, 3, (n_vars, n_cases)).astype(np.float32)
    y = rng.uniform(-9, 9, n_cases).astype(np.float32)
    nodes, offsets, use = _sums(n_vars, copies)
    consts = np.ones(1, np.float32)
    want = []
    for v in use:
        f = X[v[-1]]
        for k in v[-2::-1]:
            f = X[k] + f
        want.append(f)
    want = np.stack(want)
    assert np.array_equal(gp.predict(nodes, offsets, consts, X, synth.MASK_2), want)
    mse = ((want.astype(np.float64) - y) ** 2).mean(axis=1)
    F = gp.evaluate(nodes, offsets, consts, X, y, 0.0, synth.MASK_2)
    np.testing.assert_allclose(F, mse, rtol=2.0 ** -21)
    R = gp.evaluate_reward(nodes, offsets, consts, X, y, 11000.0, 2)
    assert np.array_equal(R, [oracle.case_rewards(f, y, 11000.0, 2).sum() for f in want])
    S = gp.evaluate_correlation(nodes, offsets, consts, X, y, 1e4)
    ref = oracle.correlation(nodes, offsets, consts, X, y, 1e4)
    ref = ref[0] if isinstance(ref, tuple) else ref
    np.testing.assert_allclose(S, ref, rtol=1e-4, atol=1e-4)


def _edges(*at):
    v = []
    for a in at:
        a = np.float32(a)
        v += [a, np.nextafter(a, np.float32(np.inf)), np.nextafter(a, np.float32(-np.inf))]
    v += [0.0, 1e-45, 1.2e-38, 3e38, np.inf, np.nan]
    v = np.array(v, np.float32)
    return np.concatenate([v, -v])


@pytest.mark.parametrize("rare", [False, True])
def test_quotients_at_the_fast_range(rare):
    """Every pair of operands around the bounds, among themselves and each
    alone among ordinary values."""
    gp = _gp()
    rng = np.random.default_rng(3)
    a = _edges(2.0 ** -60, 2.0 ** 60, 1.0, 7.0)
    b = _edges(0.001, 2.0 ** 60, 1.0, 3.0)
    a, b = (g.ravel() for g in np.meshgrid(a, b))
    if rare:
        X = rng.uniform(1, 2, (2, 256 * a.size)).astype(np.float32)
        at = np.arange(a.size) * 256 + rng.integers(0, 256, a.size)
        X[0, at], X[1, at] = a, b
    else:
        X = np.stack([a, b])
    L = synth.LOAD
    # cells, a leaf operand, a constant operand (x1 * 1 / x0 by cells)
    progs = [[L, L | 256, synth.DIV], [L, L | 256, synth.ABS, synth.ABS, synth.DIV],
             [L | 256, L, synth.DIV]]
    nodes = np.concatenate([np.array(p, np.uint32) for p in progs])
    offsets = np.concatenate([[0], np.cumsum([len(p) for p in progs])]).astype(np.int64)
    out = gp.predict(nodes, offsets, np.ones(1, np.float32), X, synth.MASK_2)

    def div(n, d):
        with np.errstate(all="ignore"):
            return np.where(np.abs(d) <= np.float32(0.001), np.float32(1), n / d)
    want = np.stack([div(X[0], X[1]), div(X[0], np.abs(X[1])), div(X[1], X[0])])
    nan = np.isnan(want)
    assert np.array_equal(np.isnan(out), nan)
    assert np.array_equal(out.view(np.uint32)[~nan], want.view(np.uint32)[~nan])


@pytest.mark.parametrize("op", [synth.SIN, synth.COS, synth.EXP, synth.LOG, synth.SQRT])
def test_functions_do_not_depend_on_their_neighbours(op):
    """A value's result is the same among its like and alone among ordinary
    ones, whichever form the wavefront takes."""
    gp = _gp()
    rng = np.random.default_rng(int(op))
    v = _edges(2.0 ** 17, 87.0, 88.8, 104.0, 0.001, 2.0 ** -100, 2.0 ** -126, 3.0, 43.0, 3e4)
    together = np.resize(v, 256)
    alone = rng.uniform(0.5, 2, (v.size, 256)).astype(np.float32)
    at = rng.integers(0, 256, v.size)
    alone[np.arange(v.size), at] = v
    nodes = np.array([synth.LOAD, op], np.uint32)
    off = np.array([0, 2], np.int64)
    consts = np.ones(1, np.float32)
    a = gp.predict(nodes, off, consts, together[None, :], synth.MASK_2)[0, :v.size]
    b = gp.predict(nodes, off, consts, alone.reshape(1, -1), synth.MASK_2)[0]
    b = b.reshape(alone.shape)[np.arange(v.size), at]
    nan = np.isnan(a)
    assert np.array_equal(np.isnan(b), nan)
    assert np.array_equal(a.view(np.uint32)[~nan], b.view(np.uint32)[~nan])


@pytest.mark.parametrize("length", [3, 63, 64, 65, 127, 128, 129, 200])
def test_full_table_around_a_chunk(length):
    """Stack moves and held variables whose programs end around the staging's
    64-node chunks, bit for bit against the oracle's float32 arithmetic (the
    commands that are correctly rounded)."""
    gp = _gp()
    rng = np.random.default_rng(length)
    pop = synth.sample_gcl_programs(rng, np.full(70, length), 4, p_pow=0.0,
                                    unary=(synth.ABS, synth.SQUARE, synth.SIGN))
    X = rng.uniform(-2, 2, (4, 130)).astype(np.float32)
    consts = pop.consts if pop.consts.size else np.ones(1, np.float32)
    out = gp.predict(pop.nodes, pop.offsets, consts, X, gp.GP_ALL_OPS)
    want = np.stack([oracle.program_outputs(pop.nodes[pop.offsets[p]:pop.offsets[p + 1]], consts, X,
                                            allowed_mask=gp.GP_ALL_OPS, mode=oracle.M32E)
                     for p in range(70)]).astype(np.float32)
    nan = np.isnan(want)
    assert np.array_equal(np.isnan(out), nan)
    assert np.array_equal(out.view(np.uint32)[~nan], want.view(np.uint32)[~nan])


@pytest.mark.parametrize("power", [1, 2, 3, 8])
@pytest.mark.parametrize("M", [10000.0, -7.0, 2.0 ** 21, 2.0 ** 21 + 1, 2.0 ** 24])
def test_rewards_at_the_fast_range(power, M):
    """Ratios of values around the bounds of the reward's fast form, among
    themselves and alone among ordinary values, signs mixed: integers, exact."""
    gp = _gp()
    rng = np.random.default_rng(power)
    v = _edges(2.0 ** -10, 2.0 ** -60, 2.0 ** 60, 1.0, 3.0)
    a, b = (g.ravel() for g in np.meshgrid(v, v))
    o = rng.uniform(-4, 4, 256 * a.size).astype(np.float32)
    y = rng.uniform(-4, 4, o.size).astype(np.float32)
    at = np.arange(a.size) * 256 + rng.integers(0, 256, a.size)
    o[at], y[at] = a, b
    nodes, off = np.array([synth.LOAD], np.uint32), np.array([0, 1], np.int64)
    for x, t in ((a, b), (o, y), (o[1:256], y[1:256])):
        R = gp.evaluate_reward(nodes, off, np.ones(1, np.float32), x[None, :], t, M, power)
        assert R[0] == oracle.case_rewards(x, t, M, power).sum()


@pytest.mark.parametrize("n", [1, 2, 255, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("S", [1, 2, 9, 10, 99, 100, 255, 256, 257])
def test_ranking_with_small_and_large_samples(n, S):
    """Bands, children and the sorted sample on both sides of the sample size
    that one kernel sorts and of a workgroup's individuals, with ties,
    infinities and NaN: exact, against the ranking oracle."""
    import torch
    from oracle import ranking
    gp = _gp()
    rng = np.random.default_rng(1000 * n + S)
    f = np.round(rng.normal(0, 3, n), 1)
    f[rng.random(n) < 0.1] = np.nan
    f[rng.random(n) < 0.1] = np.inf
    ft = torch.from_numpy(f).cuda()
    band = torch.empty(n, dtype=torch.int32, device="cuda")
    ch = torch.empty(n, dtype=torch.float32, device="cuda")
    keys = torch.empty(S, dtype=torch.float64, device="cuda")
    for higher in (False, True):
        gp.gp_mc_rank(ft, higher, 77, band, ch, keys, sample_size=S)
        want = ranking.mc_rank(f, higher, 77, S)
        assert np.array_equal(band.cpu().numpy(), want[0])
        assert np.array_equal(ch.cpu().numpy(), want[1])
        assert np.array_equal(keys.cpu().numpy(), want[2])


def test_the_widest_datasets():
    """158 variables are the most a score takes (a sub-tile of every row fills
    the LDS), 159 the most outputs take."""
    gp = _gp()
    rng = np.random.default_rng(4)
    X = rng.uniform(-3, 3, (159, 700)).astype(np.float32)
    y = rng.uniform(-9, 9, 700).astype(np.float32)
    consts = np.ones(1, np.float32)
    for n_vars in (158, 159):
        nodes, offsets, use = _sums(n_vars, 2)
        want = []
        for v in use:
            f = X[v[-1]]
            for k in v[-2::-1]:
                f = X[k] + f
            want.append(f)
        want = np.stack(want)
        assert np.array_equal(gp.predict(nodes, offsets, consts, X[:n_vars], synth.MASK_2), want)
        if n_vars == 158:
            F = gp.evaluate(nodes, offsets, consts, X[:158], y, 0.0, synth.MASK_2)
            np.testing.assert_allclose(F, ((want.astype(np.float64) - y) ** 2).mean(axis=1), rtol=2.0 ** -21)
            R = gp.evaluate_reward(nodes, offsets, consts, X[:158], y, 11000.0, 1)
            assert np.array_equal(R, [oracle.case_rewards(f, y, 11000.0, 1).sum() for f in want])
