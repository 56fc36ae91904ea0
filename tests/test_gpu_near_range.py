"""The near field of mixed plans where pairs, cells or moments differ by many
powers of two: each dipole's own error against the direct sum.

Bar: 1e-6 of the sum of the contributions' magnitudes, 2 |m_j| / r_ij^3 over the
sources j of a dipole.  A contribution takes a dozen FP32 roundings, 12 x 2^-24 =
7e-7 at worst, and the two FP16 numbers that stand for each of its factors add
2^-24 each; the positions are exact to 2^-48 of a cell side, and the cases are
small enough for every pair to be in the near field.
"""
import numpy as np
import pytest

from paper_0810_0233_amd import ccfmm, inputs

pytestmark = pytest.mark.gpu
BAR = 1e-6


@pytest.fixture(scope="module")
def ref():
    import oracle

    return oracle


def run(pos, m, **kw):
    pl = ccfmm.Plan.create(pos, ccfmm.params(max_batch=m.shape[0], precision=ccfmm.PREC_MIXED, **kw))
    assert pl.info()["n_m2l_pairs"] == 0  # near field only
    return pl.eval(m)


def worst(ref, H, pos, m):
    """Largest error of a dipole over the magnitude of its contributions."""
    r2 = np.zeros((pos.shape[0], pos.shape[0]))
    for a in range(3):
        r2 += (pos[:, None, a] - pos[None, :, a]) ** 2
    inv3 = np.where(r2 > 0, r2, np.inf) ** -1.5
    S = inv3 @ (2.0 * np.linalg.norm(m, axis=1))
    err = np.linalg.norm(H - ref.bruteforce(pos, m), axis=1)
    assert np.isfinite(H).all()
    return float((err[S > 0] / S[S > 0]).max())


# A dipole beside a much closer one that has no moment, or next to none: the
# field is that of the others.  One cell side is 1/2 (8 cells, all of them near).
@pytest.mark.parametrize("nb", [2, 3, 16, 32])
@pytest.mark.parametrize("gap", [1e-1, 1e-2, 1e-3, 1e-4, 1e-6, 1e-7])
def test_close_partner_without_moment(ref, gap, nb):
    rng = np.random.default_rng(7)
    n = 150
    a = rng.random((n, 3))
    d = rng.standard_normal((n, 3))
    pos = np.concatenate([a, a + 0.5 * gap * d / np.linalg.norm(d, axis=1)[:, None]]).clip(0, 1)
    m = np.stack([inputs.random_moments(2 * n, 30 + b) for b in range(nb)])
    m[0, n:] = 0.0
    m[1, n:] *= 1e-9
    if nb > 2:
        m[nb - 1, n:] *= np.exp2(-rng.integers(0, 20, n))[:, None]
    H = run(pos, m, order=3, theta=0.5, leaf_target=2 * n / 8.0, box=(np.zeros(3), np.ones(3)))
    for b in sorted({0, 1, nb - 1}):
        e = worst(ref, H[b], pos, m[b])
        print("case gap=%g nb=%d b=%d" % (gap, nb, b), e, flush=True)
        assert e <= BAR


# gaps of every size at once: several separate ranges of 1/r^3 in one step
@pytest.mark.parametrize("nb", [3, 16, 32])
def test_gaps_of_every_size(ref, nb):
    rng = np.random.default_rng(8)
    gap = np.repeat(10.0 ** -np.arange(0.5, 7.0, 0.25), 6)
    n = gap.size
    centre = rng.random((6, 3)) * 0.8 + 0.1
    d = rng.standard_normal((n, 3))
    pos = centre[np.arange(n) % 6] + gap[:, None] * d / np.linalg.norm(d, axis=1)[:, None]
    pos = np.concatenate([pos, centre]).clip(0, 1)
    n = pos.shape[0]
    m = np.stack([inputs.random_moments(n, 60 + b) for b in range(nb)])
    r = np.concatenate([gap, np.full(6, 1e-7)])
    m[0, r < 1e-2] = 0.0
    m[1, r < 1e-4] = 0.0
    m[2] *= (r ** 3)[:, None]  # every shell gives the centre the same
    H = run(pos, m, order=3, theta=0.5, leaf_target=n / 2.0, box=(np.zeros(3), np.ones(3)))
    for b in sorted({0, 1, 2, nb - 1}):
        e = worst(ref, H[b], pos, m[b])
        print("case nb=%d b=%d" % (nb, b), e, flush=True)
        assert e <= BAR


# Flat and long cells (a sheet, a rod) and a small opening angle: near cells that
# lie far away in units of the smallest side.  One configuration holds a single
# moment.  Outside the adjacent cells a position is rounded in the other cell's
# frame, at up to twice the separation r: 2^-24 of it in three coordinates and the
# fourth power of 1/r, 4 sqrt(3) 2^-24 x 2 = 8e-7 more.
@pytest.mark.parametrize("nb", [3, 16, 32])
@pytest.mark.parametrize("sides,levels,theta", [((8.0, 8.0, 1e-4), 6, 0.1), ((8.0, 8.0, 0.03), 6, 0.1),
                                                ((64.0, 0.02, 1.0), 6, 0.02), ((32.0, 32.0, 32.0), 9, 0.08),
                                                ((128.0, 1.0, 1.0), 7, 0.01)])
def test_far_near_cells(ref, sides, levels, theta, nb):
    rng = np.random.default_rng(9)
    n = 600
    pos = rng.random((n, 3)) * np.array(sides)
    m = np.stack([inputs.random_moments(n, 90 + b) for b in range(nb)])
    m[1, 1:] = 0.0
    H = run(pos, m, order=2, theta=theta, leaf_target=n / 2.0 ** levels, box=(np.zeros(3), np.array(sides)))
    for b in (0, 1, nb - 1):
        e = worst(ref, H[b], pos, m[b])
        print("case sides=%s nb=%d b=%d" % (sides, nb, b), e, flush=True)
        assert e <= 2 * BAR


# separations down to where 1/r^3 leaves FP32 (positions that FP32 pairs hold exactly)
@pytest.mark.parametrize("nb", [1, 3, 16, 32])
@pytest.mark.parametrize("power", [-30, -37, -39, -41])
def test_smallest_separations(ref, power, nb):
    rng = np.random.default_rng(10)
    n = 40
    a = rng.permutation(np.array(np.meshgrid(*[np.arange(1, 64, 9)] * 3)).reshape(3, -1).T)[:n] / 64.0
    pos = np.concatenate([a, a + np.array([2.0 ** power, 0.0, 2.0 ** (power - 1)])])
    m = np.stack([inputs.random_moments(2 * n, 70 + b) for b in range(nb)])
    H = run(pos, m, order=3, theta=0.5, leaf_target=2.0 * n, box=(np.zeros(3), np.ones(3)))
    for b in sorted({0, nb - 1}):
        e = worst(ref, H[b], pos, m[b])
        print("case power=%d nb=%d b=%d" % (power, nb, b), e, flush=True)
        assert e <= BAR


# Moments of very different size, the small ones in close pairs whose field is
# their own, and two configurations without such a spread beside them.
@pytest.mark.parametrize("nb", [3, 12, 16, 40])
@pytest.mark.parametrize("power", [-27, -29, -45, -60])
def test_moment_spread(ref, power, nb):
    rng = np.random.default_rng(11)
    n = 100
    gap = 0.3 * 2.0 ** (power / 3.0)
    a = rng.random((n, 3)) * np.array([0.5, 1.0, 1.0])
    d = rng.standard_normal((n, 3))
    pos = np.concatenate([a, a + 0.5 * gap * d / np.linalg.norm(d, axis=1)[:, None], [[0.99, 0.5, 0.5]]]).clip(0, 1)
    m = np.stack([inputs.random_moments(2 * n + 1, 40 + b) for b in range(nb)])
    for b in (0, nb // 2):
        m[b, :-1] *= 2.0 ** power
    H = run(pos, m, order=3, theta=0.5, leaf_target=(2 * n + 1) / 8.0, box=(np.zeros(3), np.ones(3)))
    for b in (0, nb // 2, nb - 1):
        e = worst(ref, H[b], pos, m[b])
        print("case power=%d nb=%d b=%d" % (power, nb, b), e, flush=True)
        assert e <= BAR
    H2 = run(pos, np.delete(m, [0, nb // 2], axis=0) if nb > 4 else m[1:], order=3, theta=0.5,
             leaf_target=(2 * n + 1) / 8.0, box=(np.zeros(3), np.ones(3)))
    assert np.abs(H2[-1] - H[-1]).max() <= BAR * np.abs(H[-1]).max()


# A batch is as accurate as its configurations are alone, where the near field runs
# on the FP32 vector units: rms of each dipole's error against the FP64 plan.
@pytest.mark.parametrize("order,nb", [(3, 3), (4, 8), (5, 16), (4, 32)])
def test_batch_as_accurate_as_one(order, nb):
    pos, box = inputs.ferrofluid(20000, order)
    m = np.stack([inputs.random_moments(20000, b) for b in range(nb)])

    def field(m, precision):
        kw = dict(order=order, theta=0.5, box=box, max_batch=m.shape[0])
        return ccfmm.Plan.create(pos, ccfmm.params(precision=precision, **kw)).eval(m)

    D = field(m[:3], ccfmm.PREC_FP64)
    batch = field(m, ccfmm.PREC_MIXED)[:3]
    one = np.stack([field(m[b:b + 1], ccfmm.PREC_MIXED)[0] for b in range(3)])
    e, e1 = (float(np.sqrt(np.mean(np.sum((H - D) ** 2, -1) / np.sum(D ** 2, -1)))) for H in (batch, one))
    print("case order=%d nb=%d" % (order, nb), e, e1, flush=True)
    assert e <= e1
