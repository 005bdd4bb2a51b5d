"""The per-length transform kernels (every n = 2M, 12 <= M <= 512, M =
2^a 3^b 5^c, but n = 512): all five transform types, both directions, on the contiguous
axis and on both strided axes, with ragged tiles (odd x extents, fewer lines
than a tile, a last tile that is nearly empty) and with the grid capped so
that blocks loop over tiles.  Against the Table 2 sums (<= 1e-13 relative L2,
the bound of the other transform kernels: a few roundings per FFT pass), and
against the size-generic kernel on the same fields (each within 1e-13 of the
sums, so 2e-13 of each other); FP32 through one FP32 solve."""
import numpy as np
import pytest

from gpu_util import AXIS, gpu_solve, oracle_solve, rel_l2, to_dev, to_host
from paper_1802_10323_amd import inputs

pytestmark = pytest.mark.gpu

KINDS = ("P", "NN", "DD", "ND", "DN")
LENGTHS = [n for n in inputs.smooth_sizes(24, 1024) if n != 512]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1802_10323_amd import lib
    lib()


def _cases(n, kind):
    """(shape nx ny nz, boundary pairs, role): the length-n transform along x,
    y (odd x extents above and below a tile's lines) and, periodic, z."""
    yield "x", (n, 10, 7), (kind, "P", "DD"), 0
    yield "y", (37, n, 4), ("DD", kind, "P"), 0
    yield "y", (3, n, 6), ("DN", kind, "P"), 0
    if kind == "P":
        yield "z", (21, 10, n), ("ND", "NN", "P"), 1


def _stage(shape, bcs, role, f, inverse, monkeypatch, cap=0, generic=False):
    from paper_1802_10323_amd import Plan
    monkeypatch.setenv("POISSON_GRID_CAP", str(cap))
    monkeypatch.setenv("POISSON_GENERIC_R2R", "1" if generic else "0")
    plan = Plan(*shape, 1.0, 1.0, np.ones(shape[2]), bcs)
    d = to_dev(f)
    plan.transform_stage(role, inverse, d)
    out = to_host(d)
    plan.close()
    return out


@pytest.mark.parametrize("n", LENGTHS)
def test_line_transform(n, monkeypatch):
    from oracle import transforms as tr
    rng = np.random.default_rng(n)
    for kind in KINDS:
        for axis, shape, bcs, role in _cases(n, kind):
            f = rng.uniform(-1.0, 1.0, shape[::-1])
            ref = tr.forward(f, AXIS[axis], kind)
            fwd = _stage(shape, bcs, role, f, False, monkeypatch)
            assert rel_l2(fwd, ref) <= 1e-13, (axis, kind, shape)
            assert np.array_equal(_stage(shape, bcs, role, f, False, monkeypatch, cap=1), fwd)
            gen = _stage(shape, bcs, role, f, False, monkeypatch, generic=True)
            assert rel_l2(fwd, gen) <= 2e-13, (axis, kind, shape)
            back = _stage(shape, bcs, role, ref, True, monkeypatch)
            assert rel_l2(back, f) <= 1e-13, (axis, kind, shape)
            assert np.array_equal(_stage(shape, bcs, role, ref, True, monkeypatch, cap=1), back)
            gen = _stage(shape, bcs, role, ref, True, monkeypatch, generic=True)
            assert rel_l2(back, gen) <= 2e-13, (axis, kind, shape)


@pytest.mark.parametrize("nx,ny", [(24, 1000), (50, 810), (270, 54), (300, 250), (600, 100), (1024, 90),
                                   (96, 128), (288, 384)])
@pytest.mark.parametrize("bx", KINDS)
def test_line_transform_fp32(nx, ny, bx, monkeypatch):
    """One FP32 solve (forward and backward along both axes; the last backward
    transform writes the widened FP64 solution).  Bound: four transforms of
    at most log2(1024) + 3 rounding steps per value, each 2^-24, added up; a
    random field has all wavenumbers alike, so that the elimination (FP64)
    does not raise the relative error."""
    monkeypatch.delenv("POISSON_GRID_CAP", raising=False)
    by = KINDS[(KINDS.index(bx) + nx + 1) % 5]
    prob = inputs.make_uniform(nx, ny, 9, (bx, by, "DD"), seed=nx + ny, stretch_z=1.8)
    got, _ = gpu_solve(prob, mixed=True, max_iters=1)
    assert rel_l2(got, oracle_solve(prob)) <= 4 * 13 * 2.0 ** -24
