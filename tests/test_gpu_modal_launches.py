"""The sine-mode kernels in launches of their own, on the meshes whose planes do not take them
in: z recursion, z convolution and band filter, each told by the size of the plan's z table, and
FP32 errors near rounding in every one of them.
"""
import numpy as np
import pytest

from helpers import TOL, gpu_solve, log, oracle_input, rel_l2, rel_max

pytestmark = pytest.mark.gpu

A, B, HZ = 1.2, 0.9, 0.05


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _geometry(shape, wall=(False, False)):
    return A / (shape[0] + (not wall[0])), B / (shape[1] + (not wall[1])), HZ, A, B


def _modes(shape, folds, wall=(False, False)):
    """Modes of which folds[0] x folds[1] have the same sines on the lattice."""
    return tuple(f * (n + (not w)) - 1 for f, n, w in zip(folds, shape, wall))


def _plan(shape, prec, wall, modes, **kw):
    from paper_1111_4971_amd import pipe
    return pipe.GreenPlan(*shape, *_geometry(shape, wall), precision=prec, mx=modes[0], my=modes[1], **kw)


def _table_row(plan, wall, modes):
    """Reals of the z table per mode line, from the bytes of the z pass (0: no pass of its own)."""
    i = plan.info
    lines = min(modes[0], i.nx - wall[0]) * min(modes[1], i.ny - wall[1])
    return (i.pass_bytes[2] / i.real_bytes - 2 * lines * i.nz) / lines if i.pass_bytes[2] else 0


def _exponentials(folds, prec):
    n = folds[0] * folds[1]
    n = n if n <= 2 else (n + 3) // 4 * 4
    return n if n <= (8 if prec == "fp64" else 4) else 0


ZCONV = (24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024)


def _row(folds, prec, nz):
    """Table row of the separate z pass: recursion, or the convolution's pairs."""
    ne = _exponentials(folds, prec)
    return 4 + 9 * ne if ne else 2 * (next(n for n in ZCONV if n >= nz) // 2 + 1)


def _against_padded(shape, prec, folds, wall=(False, False)):
    from paper_1111_4971_amd import pipe
    modes = _modes(shape, folds, wall)
    log("z pass %s %s folds=%s" % (prec, shape, folds))
    p = _plan(shape, prec, wall, modes)
    assert _table_row(p, wall, modes) == _row(folds, prec, shape[2])
    q = _plan(shape, prec, wall, modes, L=pipe.default_lengths(*shape, prec))
    rho = np.random.default_rng(sum(shape)).standard_normal(shape)
    got, ref = gpu_solve(p, rho), gpu_solve(q, rho)
    p.close(), q.close()
    assert rel_l2(got, ref) <= 2 * TOL[prec] and rel_max(got, ref) <= 2 * TOL[prec], rel_l2(got, ref)


# one, two, four and (FP64) eight exponentials a line, six and twelve (convolution in FP32,
# in both); 8, 12 and 16 values a lane, lines of a wave and of part of one, with and without
# a last partial lane
@pytest.mark.parametrize("folds", [(1, 1), (1, 2), (3, 1), (2, 2), (4, 2), (2, 3), (3, 4)])
@pytest.mark.parametrize("shape", [(5, 4, 500), (3, 7, 512), (4, 5, 577), (5, 3, 768), (6, 4, 769), (3, 4, 1024), (2, 3, 1001)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_long_lines_match_eq10_oracle(shape, folds, prec):
    from oracle import fourterm
    wall = (shape[2] % 2 == 0, False)
    modes = _modes(shape, folds, wall)
    log("long lines %s %s folds=%s" % (prec, shape, folds))
    p = _plan(shape, prec, wall, modes)
    assert _table_row(p, wall, modes) == _row(folds, prec, shape[2])
    rho = np.random.default_rng(sum(shape)).standard_normal(shape)
    got = gpu_solve(p, rho)
    ref = fourterm.solve(oracle_input(rho, prec), *_geometry(shape, wall), *modes, 1)
    assert rel_l2(got, ref) <= TOL[prec] and rel_max(got, ref) <= TOL[prec], rel_l2(got, ref)


@pytest.mark.parametrize("folds", [(1, 1), (2, 1), (2, 2), (2, 4), (4, 3)])
@pytest.mark.parametrize("shape", [(100, 98, 130), (66, 70, 190), (40, 36, 300), (34, 33, 257)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_short_lines_match_the_padded_transform(shape, folds, prec):
    _against_padded(shape, prec, folds, (False, shape[2] % 2 == 0))


# half lengths 48 to 128; 24 and 32 only where FP64 planes of more than 416 rows do not fit
@pytest.mark.parametrize("shape,precs", [((260, 260, 40), ("fp64", "fp32")), ((200, 201, 64), ("fp64", "fp32")),
                                         ((100, 101, 80), ("fp64", "fp32")), ((100, 98, 100), ("fp64", "fp32")),
                                         ((430, 420, 24), ("fp64",)), ((420, 418, 31), ("fp64",))])
def test_short_convolutions_match_the_padded_transform(shape, precs):
    for prec in precs:
        _against_padded(shape, prec, (3, 4) if shape[0] < 400 else (3, 3))


@pytest.mark.parametrize("nb", range(1, 17))
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_band_filters_match_the_padded_transform(nb, prec):
    """Rows that are no whole number of vectors, meshes above the limits of one launch."""
    from paper_1111_4971_amd import pipe
    shape, wall, modes = (128, 120, 171), (True, False), (240, 121)
    log("band filter %s N=%d" % (prec, nb))
    p = _plan(shape, prec, wall, modes, band=nb)
    assert _table_row(p, wall, modes) == nb + 1
    q = pipe.GreenPlan(*shape, *_geometry(shape, wall), precision=prec, mx=modes[0], my=modes[1], band=nb,
                       L=(p.info.lx, p.info.ly))
    rho = np.random.default_rng(nb).standard_normal(shape)
    got, ref = gpu_solve(p, rho), gpu_solve(q, rho)
    p.close(), q.close()
    assert rel_l2(got, ref) <= 2 * TOL[prec] and rel_max(got, ref) <= 2 * TOL[prec], rel_l2(got, ref)


# A rounding is 0.42 u of its value (u = 2^-24, root mean square over mantissas).  A chain of d
# products rounds partial sums of sqrt(k) terms, k = 1 .. d: 0.42 sqrt((d + 1) / 2) u of its sum,
# 0.9 u for the chains of 8; five levels of sums above them and the stored value add 0.94 u and
# 0.42 u, so a sine pass is at 1.4 u, and four of them with a z sum of the same at 3.0 u =
# 1.8e-7.  Half as much again is allowed; plain chains of 128 are at 3.4 u a pass, 4e-7.
@pytest.mark.parametrize("name,shape,folds,band", [
    ("planes", (30, 96, 40), (2, 2), None), ("deep planes", (161, 128, 90), (1, 1), None),
    ("deep rows", (256, 5, 33), (2, 2), None), ("streamed rows", (512, 6, 17), (1, 1), None),
    ("streamed rows", (5, 480, 12), (2, 1), None), ("recursion", (40, 40, 1024), (1, 1), None),
    ("recursion", (100, 98, 300), (2, 2), None), ("convolution", (40, 40, 1000), (3, 4), None),
    ("filter", (128, 120, 171), (1, 1), 4), ("all deep", (256, 256, 96), (1, 1), None)])
def test_fp32_error_is_near_rounding(name, shape, folds, band):
    modes = _modes(shape, folds)
    log("fp32 error: %s %s" % (name, shape))
    rho = np.abs(np.random.default_rng(sum(shape)).standard_normal(shape)).astype(np.float32)
    out = {}
    for prec in ("fp64", "fp32"):
        p = _plan(shape, prec, (False, False), modes, band=band)
        assert p.info.xtile == 0
        out[prec] = gpu_solve(p, rho)
        p.close()
    err = rel_l2(out["fp32"], out["fp64"])
    log("fp32 error %.2e" % err)
    assert err <= 4.5 * 2.0 ** -24, err


# sine passes of one and of more columns a lane: both sides of the limits at one and two
# 16-deep blocks (tiles of one column: 500, 969; 1200, 1536, 1732, 2560, 2624)
@pytest.mark.parametrize("shape", [(32, 32, 250), (30, 31, 500), (64, 64, 300), (64, 64, 384), (64, 64, 433), (64, 64, 640),
                                   (64, 64, 656)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_sine_tile_widths_match_the_padded_transform(shape, prec):
    from paper_1111_4971_amd import pipe
    modes = _modes(shape, (2, 2))
    log("tile widths %s %s" % (prec, shape))
    p = _plan(shape, prec, (False, False), modes)
    q = _plan(shape, prec, (False, False), modes, L=pipe.default_lengths(*shape, prec))
    rho = np.random.default_rng(sum(shape)).standard_normal(shape)
    got, ref = gpu_solve(p, rho), gpu_solve(q, rho)
    p.close(), q.close()
    assert rel_l2(got, ref) <= 2 * TOL[prec] and rel_max(got, ref) <= 2 * TOL[prec], rel_l2(got, ref)


@pytest.mark.parametrize("shape", [(33, 18, 40), (130, 100, 90), (300, 5, 20)])
def test_wall_nodes_are_not_read(torch_cuda, shape):
    """Charge on the walls changes nothing, whatever it is, and the potential there is 0."""
    torch = torch_cuda
    wall = (True, True)
    p = _plan(shape, "fp64", wall, _modes(shape, (2, 2), wall))
    x = torch.from_numpy(np.random.default_rng(3).standard_normal(shape)).to("cuda")
    log("wall nodes %s" % (shape,))
    ref = p.solve(x)
    x[-1], x[:, -1] = float("nan"), float("inf")
    assert torch.equal(p.solve(x), ref) and not ref[-1].any() and not ref[:, -1].any()
