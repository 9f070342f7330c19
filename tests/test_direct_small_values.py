"""GPU checks of the direct solve where a field is nearly empty: cells far from
all particles keep their value and sign, and quotients of two fields are right
wherever the divisor is not 0."""
import numpy as np
import pytest

from oracle import cgd_oracle as O

pytestmark = pytest.mark.gpu

U = np.array([0.7312, -1.9, 0.043], np.float32)


def _bed(shape, axis, seed):
    """Particles in the lower half of one axis (3: in one corner), some spread in volume; field 0 the volume,
    the others the volume times a uniform velocity."""
    rng = np.random.default_rng(seed)
    n = shape[0] * shape[1] * shape[2] // 3
    pos = rng.random((n, 3))
    if axis == 3:
        pos *= 0.25
    else:
        pos[:, axis] *= 0.5
    v = np.exp(0.3 * rng.normal(size=n)).astype(np.float32)
    vals = np.stack([v, v * U[0], v * U[1], v * U[2]])
    return pos.astype(np.float32), np.ascontiguousarray(vals)


def _allowed(ref):
    """Against the oracle: the result's one rounding to float32, and 2^-32 of
    the largest value, the most that is returned as 0 (the float64 transforms
    themselves are less than 2^-40 of it off)."""
    return 2.0 ** -24 * np.abs(ref) + (2.0 ** -32 + 2.0 ** -40) * np.abs(ref).max()


def _quotient_bound(n_plane, smallest):
    """Deposits, results and quotient are rounded to float32 once each (five
    roundings in all); the float64 transforms of both fields are 8 * 2^-53
    sqrt(n_plane) of the largest plane mean off, and the smallest divisor is
    `smallest` of that mean."""
    return 5 * 2.0 ** -24 + 2 * 8 * 2.0 ** -53 * np.sqrt(n_plane) / smallest


def _check(cgd, torch, out, n_plane, tag):
    eps = out[0].cpu().numpy()
    assert (eps >= 0).all(), tag
    assert (eps > 0).any()
    scale = float(eps.max())
    for eps_min in (1e-6 * scale, 1e-8 * scale, 0.0):
        u = cgd.velocity_from_momentum(out[0].contiguous(), out[1:].clone(), eps_min=eps_min).cpu().numpy()
        sel = eps > np.float32(eps_min)
        assert sel.any()
        tol = _quotient_bound(n_plane, eps_min / scale if eps_min else 2.0 ** -32)
        for c in range(3):
            err = np.abs(u[c][sel].astype(np.float64) / U[c] - 1).max()
            assert err <= tol, (tag, eps_min, c, err)
        assert not u[:, ~sel].any()


# FFT lengths, matrix lengths and both; steps and bandwidths that reach far and hardly at all
@pytest.mark.parametrize("shape", [(64, 40, 48), (128, 20, 16), (33, 128, 30), (24, 24, 128)])
@pytest.mark.parametrize("axis", [0, 1, 2, 3])
def test_nearly_empty_cells(gpu_lib, shape, axis):
    import torch
    cgd = gpu_lib
    mesh = cgd.HexMesh(shape, (0, 0, 0), tuple(n / 64.0 for n in shape))
    pos, vals = _bed(shape, axis, 3)
    pos = pos * np.array([n / 64.0 for n in shape], np.float32)
    p, v = torch.from_numpy(pos).cuda(), torch.from_numpy(vals).cuda()
    for bcells, steps in ((4.0, 4), (0.6, 1), (2.0, 6)):
        tag = f"thin hex {shape} axis {axis} b {bcells}h steps {steps}"
        print("case:", tag, flush=True)
        out = cgd.coarse_grain(mesh, p, v, bcells / 64.0, steps)[0]
        _check(cgd, torch, out, shape[0] * shape[1], tag)
        e0 = cgd.deposit(mesh, p, v)
        ref = O.diffuse_hex_dct(e0.cpu().numpy().astype(np.float64), (0, 0, 0), tuple(n / 64.0 for n in shape), shape,
                                bcells / 64.0, steps)
        got = out.cpu().numpy().astype(np.float64)
        for f in range(4):
            assert (np.abs(got[f] - ref[f]) <= _allowed(ref[f])).all(), (tag, f)
        one = cgd.diffuse(mesh, e0[:1].clone(), bcells / 64.0, steps)[0]
        assert torch.equal(one[0].view(torch.int32), out[0].view(torch.int32))


def test_nearly_empty_cells_batched(gpu_lib):
    import torch
    cgd = gpu_lib
    shape = (64, 40, 24)
    mesh = cgd.HexMesh(shape)
    parts = [_bed(shape, a, 5 + a) for a in (0, 1, 3)]
    off = np.concatenate([[0], np.cumsum([len(p) for p, _ in parts])]).astype(np.int64)
    pos = torch.from_numpy(np.concatenate([p for p, _ in parts])).cuda()
    vals = torch.from_numpy(np.ascontiguousarray(np.concatenate([v for _, v in parts], axis=1))).cuda()
    print("case: thin batched", flush=True)
    out = cgd.coarse_grain_batched(mesh, off, pos, vals, 0.05, 3)
    for j in range(3):
        _check(cgd, torch, out[j], shape[0] * shape[1], f"thin batched {j}")


@pytest.mark.parametrize("periodic", [(False,) * 3, (False, True, False)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_nearly_empty_cells_rect(gpu_lib, axis, periodic):
    """Widths that vary threefold: the volume-weighted transforms."""
    import torch
    cgd = gpu_lib
    shape = (48, 40, 44)
    edges = []
    for a, n in enumerate(shape):
        w = 1.0 + 2.0 * np.abs(np.arange(n) - (n - 1) / 2.0) / n
        e = np.concatenate([[0.0], np.cumsum(w)])
        e /= e[-1]
        e[-1] = 1.0
        edges.append(e)
    mesh = cgd.RectMesh(*edges, periodic=periodic)
    pos, vals = _bed(shape, axis, 9)
    if periodic[axis]:
        pos[:, axis] *= 0.5
    print(f"case: thin rect axis {axis} periodic {periodic}", flush=True)
    out = cgd.coarse_grain(mesh, torch.from_numpy(pos).cuda(), torch.from_numpy(vals).cuda(), 0.04, 3)[0]
    _check(cgd, torch, out, shape[0] * shape[1], f"thin rect {axis}")


def test_signed_fields_keep_their_small_values(gpu_lib):
    """A field with a negative value anywhere is not cut: its far values are
    the transforms' own, small and not all 0."""
    import torch
    cgd = gpu_lib
    shape = (64, 40, 128)
    mesh = cgd.HexMesh(shape, (0, 0, 0), tuple(n / 64.0 for n in shape))
    rng = np.random.default_rng(4)
    e0 = np.zeros((2, mesh.cells), np.float32)
    e0[:, : 64 * 40 * 32] = rng.random((2, 64 * 40 * 32))
    e0[1, 7] = -1.0
    print("case: signed field", flush=True)
    out = cgd.diffuse(mesh, torch.from_numpy(e0).cuda(), 1.0 / 64.0, 4)[0].cpu().numpy()
    far = out[:, 64 * 40 * 100:]
    assert (out[0] >= 0).all() and not far[0].any()
    assert far[1].any() and np.abs(far[1]).max() <= 2.0 ** -44
