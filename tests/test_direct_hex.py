"""GPU parity of the direct solve of uniform hex grids (spectral.hip): the calls
that ask for no solver statistics, against the oracle's closed form."""
import numpy as np
import pytest

from oracle import cgd_oracle as O
from paper_1409_0001_amd import inputs

pytestmark = pytest.mark.gpu


def _bound(e0, ref):
    """The vectors between the transforms are float32, rounded at most five
    times (relative error 2^-24 each, everything else in float64); the
    transforms keep the 2-norm and the gains are at most 1, so the error is
    at most 5 * 2^-24 ||e0||."""
    return 5 * 2.0 ** -24 * np.linalg.norm(e0) + 1e-30


def _field(shape, F, seed):
    rng = np.random.default_rng(seed)
    f = rng.random((F, shape[0] * shape[1] * shape[2])).astype(np.float32) ** 4
    if F > 1:
        f[1] = rng.normal(size=f.shape[1])
    return f


# FFT lengths on each axis (one block of lines and several, odd numbers of
# lines, lines of odd strides), matrix lengths at the edges of their 16-row
# tiles and of their numbers of tiles per wave, the smallest and largest of
# both, grids of two axes
@pytest.mark.parametrize("shape", [(2, 2, 2), (16, 17, 15), (31, 32, 33), (64, 65, 5), (127, 3, 9), (5, 129, 255),
                                   (257, 6, 4), (3, 4, 511), (512, 7, 6), (128, 5, 7), (9, 128, 11), (7, 5, 128),
                                   (256, 33, 3), (33, 256, 2), (3, 3, 256), (5, 512, 3), (6, 5, 512), (1024, 3, 2),
                                   (3, 1024, 2), (2, 3, 1024), (40, 1, 70), (1, 128, 20), (300, 130, 1)])
@pytest.mark.parametrize("scheme", ["be", "cn"])
def test_direct_matches_oracle(gpu_lib, shape, scheme):
    import torch
    cgd = gpu_lib
    hi = tuple(n / 64.0 for n in shape)
    print(f"case: direct {shape} {scheme}", flush=True)
    mesh = cgd.HexMesh(shape, (0, 0, 0), hi)
    e0 = _field(shape, 3, 5)
    out = cgd.diffuse(mesh, torch.from_numpy(e0).cuda(), 4 / 64.0, 3, scheme=scheme)[0].cpu().numpy()
    ref = O.diffuse_hex_dct(e0.astype(np.float64), (0, 0, 0), hi, shape, 4 / 64.0, 3, scheme=scheme)
    for f in range(3):
        assert np.linalg.norm(out[f].astype(np.float64) - ref[f]) <= _bound(e0[f], ref[f]), f


@pytest.mark.parametrize("shape", [(128, 20, 9), (50, 20, 9)])
@pytest.mark.parametrize("steps,bcells", [(1, 0.5), (1, 24.0), (7, 3.0), (64, 8.0)])
def test_direct_step_sizes_alignment_and_field_count(gpu_lib, shape, steps, bcells):
    """Few and many steps, small and large; a field that is only 4-byte
    aligned, and the same field alone and among others, give the same bits."""
    import torch
    cgd = gpu_lib
    hi = tuple(n / 64.0 for n in shape)
    mesh = cgd.HexMesh(shape, (0, 0, 0), hi)
    e0 = _field(shape, 4, 6)
    print(f"case: direct {shape} steps {steps} b {bcells}h", flush=True)
    out = cgd.diffuse(mesh, torch.from_numpy(e0).cuda(), bcells / 64.0, steps)[0].cpu().numpy()
    ref = O.diffuse_hex_dct(e0.astype(np.float64), (0, 0, 0), hi, shape, bcells / 64.0, steps)
    for f in range(4):
        assert np.linalg.norm(out[f].astype(np.float64) - ref[f]) <= _bound(e0[f], ref[f]), f
    n = mesh.cells
    buf = torch.empty(n + 1, device="cuda")
    one = buf[1:].view(1, n)
    one.copy_(torch.from_numpy(e0[2:3]))
    cgd.diffuse(mesh, one, bcells / 64.0, steps)
    assert np.array_equal(one.cpu().numpy()[0].view(np.uint32), out[2].view(np.uint32))


@pytest.mark.parametrize("shape", [(128, 16, 12), (30, 20, 10)])
def test_direct_hands_what_it_cannot_carry_to_cg(gpu_lib, shape, monkeypatch):
    """A field whose transform overflows float32 (the larger grid's) is solved by CG as before,
    one that is not finite is a breakdown as before, and the fields beside
    them are solved."""
    import torch
    cgd = gpu_lib
    hi = tuple(n / 64.0 for n in shape)
    mesh = cgd.HexMesh(shape, (0, 0, 0), hi)
    e0 = _field(shape, 3, 7)
    e0[0] = 1.0e37 * (1.0 + 0.5 * e0[0])
    # the largest value stored between passes: the mean over x and y times sqrt(nx ny)
    beyond = float(e0[0].astype(np.float64).mean()) * np.sqrt(shape[0] * shape[1]) > np.finfo(np.float32).max
    assert beyond == (shape[0] == 128)
    print(f"case: direct fallback {shape}", flush=True)
    f = torch.from_numpy(e0).cuda()
    cgd.diffuse(mesh, f, 1 / 64.0, 2)
    out = f.cpu().numpy().astype(np.float64)
    ref = O.diffuse_hex_dct(e0.astype(np.float64), (0, 0, 0), hi, shape, 1 / 64.0, 2)
    for k in range(3):
        assert np.linalg.norm(out[k] - ref[k]) <= 1e-5 * np.linalg.norm(ref[k]), k
    monkeypatch.setenv("CGD_NO_DIRECT", "1")
    cg = torch.from_numpy(e0).cuda()
    cgd.diffuse(mesh, cg, 1 / 64.0, 2)
    assert torch.equal(cg[0].view(torch.int32), f[0].view(torch.int32)) == beyond
    monkeypatch.delenv("CGD_NO_DIRECT")
    for bad in (float("nan"), float("inf")):
        g = torch.from_numpy(e0[1:]).cuda()
        g[0, 5] = bad
        with pytest.raises(cgd.CgdError) as e:
            cgd.diffuse(mesh, g, 4 / 64.0, 3)
        assert e.value.status == -5
        want = O.diffuse_hex_dct(e0[2:].astype(np.float64), (0, 0, 0), hi, shape, 4 / 64.0, 3)
        assert np.linalg.norm(g[1].cpu().numpy().astype(np.float64) - want[0]) <= _bound(e0[2], want)


def test_what_stays_with_cg(gpu_lib):
    """Statistics, a tolerance below the default, a start from a guess, plain
    CG and few iterations are the CG's, whose own bits they keep; the rest
    agrees with them to the stopping rule."""
    import torch
    cgd = gpu_lib
    shape = (64, 24, 20)
    mesh = cgd.HexMesh(shape)
    p = inputs.uniform_bed(inputs.HexBox((0, 0, 0), (1, 1, 1), shape), 20_000, 2, seed=3, diam=0.01)
    pos, vals = torch.from_numpy(p.pos).cuda(), torch.from_numpy(p.values).cuda()
    b, steps = 0.06, 3
    cg, st = cgd.coarse_grain(mesh, pos, vals, b, steps, stats=True)
    assert st.status == 0 and all(i >= 1 for row in st.iters for i in row)
    fast = cgd.coarse_grain(mesh, pos, vals, b, steps)[0]
    assert not torch.equal(fast, cg)
    assert float((fast - cg).norm() / cg.norm()) <= 1e-5
    again = cgd.coarse_grain(mesh, pos, vals, b, steps)[0]
    assert torch.equal(again.view(torch.int32), fast.view(torch.int32))
    tight, st7 = cgd.coarse_grain(mesh, pos, vals, b, steps, rtol=1e-7, stats=True)
    assert torch.equal(cgd.coarse_grain(mesh, pos, vals, b, steps, rtol=1e-7)[0].view(torch.int32),
                       tight.view(torch.int32))
    plain = cgd.coarse_grain(mesh, pos, vals, b, steps, precond=1, stats=True)[0]
    assert torch.equal(cgd.coarse_grain(mesh, pos, vals, b, steps, precond=1)[0].view(torch.int32),
                       plain.view(torch.int32))
    few, st1 = cgd.coarse_grain(mesh, pos, vals, b, steps, max_iter=1, stats=True)
    assert st1.status == 1
    assert torch.equal(cgd.coarse_grain(mesh, pos, vals, b, steps, max_iter=1)[0].view(torch.int32),
                       few.view(torch.int32))


@pytest.mark.parametrize("F,counts", [(1, [5000, 0, 1, 9000]), (3, [4000] * 7)])
def test_direct_batched(gpu_lib, F, counts):
    """The batched call without statistics: every snapshot the bits of its
    own cgd_coarse_grain; non-finite particles reported as before."""
    import torch
    cgd = gpu_lib
    shape = (48, 40, 36)
    mesh = cgd.HexMesh(shape)
    box = inputs.HexBox((0, 0, 0), (1, 1, 1), shape)
    parts = [inputs.uniform_bed(box, n, F, seed=10 + j, diam=0.01) for j, n in enumerate(counts)]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    pos = torch.from_numpy(np.concatenate([p.pos for p in parts])).cuda()
    vals = torch.from_numpy(np.ascontiguousarray(np.concatenate([p.values for p in parts], axis=1))).cuda()
    print(f"case: direct batched F={F} {counts}", flush=True)
    out = cgd.coarse_grain_batched(mesh, off, pos, vals, 0.08, 3)
    for j in range(len(counts)):
        s = slice(int(off[j]), int(off[j + 1]))
        one = cgd.coarse_grain(mesh, pos[s].contiguous(), vals[:, s].contiguous(), 0.08, 3)[0]
        assert torch.equal(one.view(torch.int32), out[j].view(torch.int32)), j
    pos[3, 1] = float("nan")
    with pytest.raises(cgd.CgdError) as e:
        cgd.coarse_grain_batched(mesh, off, pos, vals, 0.08, 3)
    assert e.value.status == -2


# near the line of the cost rule, one step: FFT and matrix lengths, and one that stays with the CG
@pytest.mark.parametrize("shape", [(120, 120, 120), (128, 100, 90), (300, 100, 60)])
def test_route_does_not_depend_on_the_number_of_fields(gpu_lib, shape):
    """A field alone, among four and in a batch: the same bits."""
    import torch
    cgd = gpu_lib
    mesh = cgd.HexMesh(shape)
    p = inputs.uniform_bed(inputs.HexBox((0, 0, 0), (1, 1, 1), shape), 60_000, 4, seed=8, diam=0.01)
    pos, vals = torch.from_numpy(p.pos).cuda(), torch.from_numpy(p.values).cuda()
    print(f"case: route {shape}", flush=True)
    four = cgd.coarse_grain(mesh, pos, vals, 0.03, 1)[0]
    off = np.array([0, 60_000, 120_000], np.int64)
    batch = cgd.coarse_grain_batched(mesh, off, torch.cat([pos, pos]), torch.cat([vals, vals], dim=1).contiguous(), 0.03, 1)
    for f in range(4):
        one = cgd.coarse_grain(mesh, pos, vals[f:f + 1].contiguous(), 0.03, 1)[0]
        assert torch.equal(one[0].view(torch.int32), four[f].view(torch.int32)), f
    if shape[0] != 300:  # (the batched CG's sums differ from the single call's, as before)
        assert torch.equal(batch[0].view(torch.int32), four.view(torch.int32))
        assert torch.equal(batch[1].view(torch.int32), four.view(torch.int32))


@pytest.mark.parametrize("kind", ["overflow", "infinite"])
def test_batched_hands_over_single_right_hand_sides(gpu_lib, kind):
    """A snapshot with one field that the transforms cannot carry: every field
    of the batch, that one and the healthy ones, is the bits of its own
    cgd_coarse_grain, and the status is its status."""
    import torch
    cgd = gpu_lib
    shape, n = (128, 16, 12), 40_000
    mesh = cgd.HexMesh(shape)
    box = inputs.HexBox((0, 0, 0), (1, 1, 1), shape)
    parts = [inputs.uniform_bed(box, n, 2, seed=20 + j, diam=0.01) for j in range(3)]
    pos = torch.from_numpy(np.concatenate([p.pos for p in parts])).cuda()
    vals = np.ascontiguousarray(np.concatenate([p.values for p in parts], axis=1))
    # mean density 1.2e37: finite, its x-y modes are not (1.2e37 * sqrt(128 * 16)); or an infinite density
    vals[1, n:2 * n] = np.float32(1.2e37 / n if kind == "overflow" else 3e38)
    vals = torch.from_numpy(vals).cuda()
    off = np.array([0, n, 2 * n, 3 * n], np.int64)
    print(f"case: batched hand-over {kind}", flush=True)

    def call(f):
        try:
            f()
            return 0, ""
        except cgd.CgdError as e:
            return e.status, str(e)

    out = torch.full((3, 2, mesh.cells), -1.0, device="cuda")
    status, message = call(lambda: cgd.coarse_grain_batched(mesh, off, pos, vals, 0.01, 3, fields=out))
    want = 0
    for j in range(3):
        s = slice(j * n, (j + 1) * n)
        one = torch.full((2, mesh.cells), -1.0, device="cuda")
        st, _ = call(lambda: cgd.coarse_grain(mesh, pos[s].contiguous(), vals[:, s].contiguous(), 0.01, 3, field=one))
        want = want or st
        if kind == "overflow" or j != 1:
            assert torch.equal(one.view(torch.int32), out[j].view(torch.int32)), j
        else:
            assert torch.equal(one[0].view(torch.int32), out[j][0].view(torch.int32))
    assert status == want == (0 if kind == "overflow" else -5)
    if kind == "infinite":
        assert "right-hand side 3" in message


def test_direct_passes_are_timed(gpu_lib):
    """With timing enabled, the transform passes are recorded: two along x,
    three along the other axes, with the bytes they move."""
    import torch
    cgd = gpu_lib
    shape = (128, 40, 33)
    mesh = cgd.HexMesh(shape)
    e0 = torch.from_numpy(_field(shape, 2, 5)).cuda()
    cgd.timing_enable(mesh, True)
    for _ in range(2):
        cgd.diffuse(mesh, e0.clone(), 0.05, 3)
    cgd.timing_enable(mesh, False)
    cgd.diffuse(mesh, e0.clone(), 0.05, 3)
    t = cgd.timing_read(mesh, reset=True)
    assert t["cg_sweep1"][0] == 4 and t["cg_sweep2"][0] == 6
    assert t["cg_sweep1"][1] > 0 and t["cg_sweep2"][1] > 0
    assert t["cg_sweep1"][2] == 24.0 * mesh.cells and t["cg_sweep2"][2] == 32.0 * mesh.cells
    assert not any(v[0] for k, v in t.items() if k not in ("cg_sweep1", "cg_sweep2"))


@pytest.mark.parametrize("switch", ["CGD_HEX_PRECOND_DEG=4", "CGD_HEX_LDS_ZC=4", "CGD_HEX_DIR=0", "CGD_HEX_DIR_NW=16",
                                    "CGD_HEX_DIR_ZC=4", "CGD_HEX_NO_SWAP=1", "CGD_HEX_TILE=2,4", "CGD_NO_BUDGET=1"])
def test_switches_of_the_cg_reach_it(gpu_lib, switch, monkeypatch):
    """A call without statistics under a switch of the CG: the CG's bits."""
    import torch
    cgd = gpu_lib
    shape = (64, 24, 20)
    mesh = cgd.HexMesh(shape)
    e0 = torch.from_numpy(_field(shape, 1, 9)).cuda()
    print(f"case: switch {switch}", flush=True)
    direct = cgd.diffuse(mesh, e0.clone(), 0.06, 3)[0]
    monkeypatch.setenv(*switch.split("="))
    got = cgd.diffuse(mesh, e0.clone(), 0.06, 3)[0]
    want = cgd.diffuse(mesh, e0.clone(), 0.06, 3, stats=True)[0]
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert not torch.equal(got, direct)


# more cells than a group of fields takes at once (16.7M): fields in two groups, an even and an odd number of cells
@pytest.mark.parametrize("shape,F", [((256, 256, 64), 6), ((255, 257, 65), 5)])
def test_fields_in_several_groups(gpu_lib, shape, F):
    import torch
    cgd = gpu_lib
    mesh = cgd.HexMesh(shape)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    e0 = torch.rand((F, mesh.cells), device="cuda", generator=g) ** 4
    e0[1] -= 0.5
    print(f"case: groups {shape} F={F}", flush=True)
    out = cgd.diffuse(mesh, e0.clone(), 0.02, 3)[0]
    assert not torch.equal(out[0], e0[0])
    for f in range(F):
        one = cgd.diffuse(mesh, e0[f:f + 1].clone(), 0.02, 3)[0]
        assert torch.equal(one[0].view(torch.int32), out[f].view(torch.int32)), f
    n = 30_000
    pos = torch.rand((3 * n, 3), device="cuda", generator=g)
    vals = torch.rand((2, 3 * n), device="cuda", generator=g)
    off = np.array([0, n, 2 * n, 3 * n], np.int64)
    batch = cgd.coarse_grain_batched(mesh, off, pos, vals, 0.02, 3)
    for j in range(3):
        s = slice(j * n, (j + 1) * n)
        one = cgd.coarse_grain(mesh, pos[s].contiguous(), vals[:, s].contiguous(), 0.02, 3)[0]
        assert torch.equal(one.view(torch.int32), batch[j].view(torch.int32)), j


@pytest.mark.parametrize("shape", [(128, 40, 33), (50, 30, 20)])
def test_other_streams(gpu_lib, shape):
    """The first call (which makes the tables) on one stream, others on
    another and on the default one, each after its input on that stream."""
    import torch
    cgd = gpu_lib
    e0 = torch.from_numpy(_field(shape, 2, 5))
    want = cgd.diffuse(cgd.HexMesh(shape), e0.cuda(), 0.05, 3)[0]
    mesh = cgd.HexMesh(shape)
    host = e0.pin_memory()
    torch.cuda.synchronize()
    for s in (torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.default_stream()):
        with torch.cuda.stream(s):
            f = host.to("cuda", non_blocking=True) * 1.0
            got = cgd.diffuse(mesh, f, 0.05, 3)[0]
            same = torch.equal(got.view(torch.int32), want.view(torch.int32))
        assert same
