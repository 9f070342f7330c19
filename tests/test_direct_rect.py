"""GPU parity of the direct solve on rectilinear grids (one diffusivity on a
box of cells, 0 elsewhere), against the oracle's sparse direct solve, and what
stays with the CG."""
import numpy as np
import pytest

from oracle import cgd_oracle as O

pytestmark = pytest.mark.gpu


def _edges(n, lo, length, how, seed):
    rng = np.random.default_rng(seed)
    if how == "even":
        w = np.ones(n)
    elif how == "mirror":  # finer at the ends, its own mirror image
        w = 1.1 ** -np.abs(np.arange(n) - (n - 1) / 2.0)
    elif how == "geometric":
        w = 1.05 ** np.arange(n)
    else:
        w = 0.3 + rng.random(n)
    e = lo + np.concatenate(([0.0], np.cumsum(w))) * (length / w.sum())
    e[-1] = lo + length
    return e


# widths per axis, periodic axes, cut: cells of diffusivity 0 at the lower and
# upper end of each axis (None: no diffusivity given), and the constant elsewhere
CASES = [
    ((12, 9, 7), ("even", "mirror", "geometric"), (False,) * 3, None),
    ((20, 17, 15), ("random", "geometric", "random"), (False,) * 3, ((0, 0), (0, 0), (0, 0), 0.37)),
    ((33, 16, 18), ("mirror", "even", "mirror"), (True, True, False), None),
    ((16, 2, 9), ("even", "even", "geometric"), (True, True, False), None),
    ((7, 3, 2), ("mirror", "mirror", "even"), (True, True, True), None),
    ((24, 10, 11), ("mirror", "even", "random"), (False,) * 3, ((4, 4), (0, 0), (0, 0), 1.0)),
    ((24, 10, 11), ("mirror", "even", "random"), (False,) * 3, ((5, 2), (1, 3), (2, 0), 2.5)),
    ((130, 6, 5), ("even", "even", "even"), (False,) * 3, ((1, 1), (0, 2), (0, 0), 1.0)),   # FFT rows at an odd start
    ((130, 7, 128), ("mirror", "even", "even"), (False, True, False), ((0, 0), (0, 0), (0, 0), 1.0)),
    ((9, 40, 1), ("geometric", "mirror", "even"), (False, True, False), None),
    ((9, 1, 40), ("geometric", "even", "mirror"), (False, True, False), ((1, 1), (0, 0), (3, 3), 1.0)),
    ((12, 8, 10), ("even", "even", "even"), (True, False, False), ((2, 1), (0, 0), (0, 0), 1.0)),  # the gap opens the ring
    ((256, 3, 4), ("random", "even", "even"), (False,) * 3, None),                          # the longest full matrix
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("scheme", ["be", "cn"])
def test_direct_rect_matches_oracle(gpu_lib, case, scheme):
    """All errors are roundings of the float32 vectors between the passes (at
    most five, 2^-24 each), in the norm weighted by the cell volumes, in which
    the transforms are orthonormal and the gains at most 1.  Cells without
    diffusivity keep their bits."""
    import torch
    cgd = gpu_lib
    shape, how, per, cut = CASES[case]
    e = [_edges(shape[a], 0.2 * a, shape[a] / 24.0, how[a], 7 + a) for a in range(3)]
    D = None
    if cut is not None:
        D = np.zeros(shape[::-1], np.float32)
        s = tuple(slice(cut[a][0], shape[a] - cut[a][1]) for a in (2, 1, 0))
        D[s] = cut[3]
        D = D.ravel()
    print(f"case: direct rect {shape} {how} periodic {per} cut {cut} {scheme}", flush=True)
    mesh = cgd.RectMesh(*e, diffusivity=D, periodic=per)
    rng = np.random.default_rng(case)
    e0 = (rng.random((2, mesh.cells)) ** 3).astype(np.float32)
    e0[1] -= 0.3
    b, steps = 0.1, 3
    f = torch.from_numpy(e0).cuda()
    out = cgd.diffuse(mesh, f, b, steps, scheme=scheme)[0].cpu().numpy()
    ref = O.diffuse_rect(e0.astype(np.float64), e, b, steps, diffusivity=D, solver="direct", scheme=scheme, periodic=per)
    w = np.sqrt(O.rect_volumes(e))
    for k in range(2):
        err = np.linalg.norm(w * (out[k].astype(np.float64) - ref[k]))
        assert err <= 5 * 2.0 ** -24 * np.linalg.norm(w * e0[k]), (k, err / np.linalg.norm(w * e0[k]))
        if D is not None:
            assert np.array_equal(out[k][D == 0].view(np.uint32), e0[k][D == 0].view(np.uint32))


def test_rect_that_stays_with_cg(gpu_lib, monkeypatch):
    """Diffusivities that vary, gaps inside, statistics and tight tolerances:
    the bits of the CG (CGD_NO_DIRECT); a constant one is solved directly."""
    import torch
    cgd = gpu_lib
    shape = (20, 12, 10)
    e = [_edges(shape[a], 0.0, 1.0, "mirror", a) for a in range(3)]
    rng = np.random.default_rng(2)
    e0 = torch.from_numpy(rng.random((1, 2400)).astype(np.float32)).cuda()
    vary = np.broadcast_to(0.5 + 0.1 * np.arange(20, dtype=np.float32), shape[::-1]).ravel().copy()
    gap = np.ones(shape[::-1], np.float32)
    gap[:, :, 9] = 0.0
    some = (0.5 + rng.random(2400)).astype(np.float32)  # no product of per-axis factors
    for name, D, direct in (("vary", vary, False), ("gap", gap.ravel(), False), ("any", some, False),
                            ("one", None, True)):
        print(f"case: rect route {name}", flush=True)
        mesh = cgd.RectMesh(*e, diffusivity=D)
        got = cgd.diffuse(mesh, e0.clone(), 0.2, 2)[0]
        with_stats = cgd.diffuse(mesh, e0.clone(), 0.2, 2, stats=True)[0]
        tight = cgd.diffuse(mesh, e0.clone(), 0.2, 2, rtol=1e-7)[0]
        monkeypatch.setenv("CGD_NO_DIRECT", "1")
        cg = cgd.diffuse(mesh, e0.clone(), 0.2, 2)[0]
        cg_tight = cgd.diffuse(mesh, e0.clone(), 0.2, 2, rtol=1e-7)[0]
        monkeypatch.delenv("CGD_NO_DIRECT")
        assert torch.equal(with_stats, cg) and torch.equal(tight, cg_tight)
        assert torch.equal(got, cg) == (not direct)
        assert float((got - cg).norm() / cg.norm()) <= 1e-5


def test_rect_not_finite(gpu_lib):
    import torch
    cgd = gpu_lib
    e = [_edges(n, 0.0, 1.0, "mirror", 1) for n in (18, 8, 6)]
    mesh = cgd.RectMesh(*e)
    f = torch.ones((2, mesh.cells), dtype=torch.float32, device="cuda")
    f[1, 3] = float("nan")
    with pytest.raises(cgd.CgdError) as err:
        cgd.diffuse(mesh, f, 0.2, 2)
    assert err.value.status == -5
    assert torch.allclose(f[0], torch.ones_like(f[0]), rtol=1e-6)


@pytest.mark.parametrize("where", [(0, 0, 0), (19, 5, 4), (5, 0, 4), (5, 5, 9), (2, 5, 4)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_rect_not_finite_outside_the_box(gpu_lib, where, bad, monkeypatch):
    """A value that is not finite in a cell without diffusivity: the CG's
    status, for its field alone."""
    import torch
    cgd = gpu_lib
    shape, cut = (20, 12, 10), ((3, 2), (1, 2), (1, 1))
    e = [_edges(n, 0.0, 1.0, "mirror", 1) for n in shape]
    D = np.zeros(shape[::-1], np.float32)
    D[tuple(slice(cut[a][0], shape[a] - cut[a][1]) for a in (2, 1, 0))] = 1.0
    mesh = cgd.RectMesh(*e, diffusivity=D.ravel())
    f = np.ones((2, mesh.cells), np.float32)
    f[1, where[0] + 20 * (where[1] + 12 * where[2])] = bad
    assert D[where[::-1]] == 0
    print(f"case: direct rect {bad} at {where}", flush=True)
    status = []
    for env in (None, "1"):
        if env:
            monkeypatch.setenv("CGD_NO_DIRECT", env)
        t = torch.from_numpy(f).cuda()
        with pytest.raises(cgd.CgdError) as err:
            cgd.diffuse(mesh, t, 0.2, 2)
        status.append(err.value.status)
        assert str(err.value).endswith(", field 1")
        if not env:  # (the CG leaves the field beside it to its own tolerance)
            assert torch.allclose(t[0], torch.ones_like(t[0]), rtol=1e-6)
    assert status == [-5, -5]


# even numbers of cells and odd, one short of and beyond a tile, FFT lengths (which a periodic axis takes as
# matrices), the longest
@pytest.mark.parametrize("n", [2, 3, 31, 33, 128, 255, 512])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_periodic_axis_of_even_cells(gpu_lib, n, axis):
    """Cosines and sines in closed form; the other axes uneven and a cosine axis."""
    import torch
    cgd = gpu_lib
    shape = [7, 6, 5]
    shape[axis] = n
    e = [_edges(shape[a], 0.1, shape[a] / 24.0, "even" if a in (axis, (axis + 1) % 3) else "random", a) for a in range(3)]
    per = tuple(a == axis for a in range(3))
    mesh = cgd.RectMesh(*e, periodic=per)
    rng = np.random.default_rng(n + axis)
    e0 = (rng.random((2, mesh.cells)) ** 3).astype(np.float32)
    e0[1] -= 0.3
    print(f"case: direct periodic {shape} axis {axis}", flush=True)
    out = cgd.diffuse(mesh, torch.from_numpy(e0).cuda(), 0.3, 3)[0].cpu().numpy()
    ref = O.diffuse_rect(e0.astype(np.float64), e, 0.3, 3, solver="direct", periodic=per)
    w = np.sqrt(O.rect_volumes(e))
    for k in range(2):
        assert np.linalg.norm(w * (out[k].astype(np.float64) - ref[k])) <= 5 * 2.0 ** -24 * np.linalg.norm(w * e0[k]), k
