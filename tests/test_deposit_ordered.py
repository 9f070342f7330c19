"""GPU deposit through the ordering pass (records kept per chunk of particles
in tile order, runs gathered by the accumulation): bit for bit the oracle's."""
import numpy as np
import pytest

from oracle import cgd_oracle as O
from paper_1409_0001_amd import inputs

pytestmark = pytest.mark.gpu


def _check(cgd, torch, shape, pos, vals, print_case):
    print(f"case: {print_case}", flush=True)
    mesh = cgd.HexMesh(shape)
    F = vals.shape[0]
    acc = torch.empty((F, mesh.cells), dtype=torch.int64, device="cuda")
    field, st = cgd.deposit(mesh, torch.from_numpy(pos).cuda(), torch.from_numpy(vals).cuda(), acc=acc, stats=True)
    ref = O.deposit_hex(pos, vals, (0, 0, 0), (1, 1, 1), shape)
    assert np.array_equal(acc.cpu().numpy(), ref["acc"])
    assert np.array_equal(field.cpu().numpy().view(np.uint32), ref["field32"].view(np.uint32))
    # (the oracle counts particles with a non-finite position; the library adds the non-finite values)
    assert st.n_dropped == ref["n_dropped"]
    assert st.n_nonfinite == ref["n_nonfinite"] + int((~np.isfinite(vals)).sum())
    assert st.frac_bits == list(ref["S"])


# chunk edges (2048 particles), a few particles, one; tiles of 64 cells and a
# ragged last one; every number of fields the records hold
@pytest.mark.parametrize("n", [1, 63, 2047, 2048, 2049, 40_000])
@pytest.mark.parametrize("F", [1, 2, 3, 4])
def test_chunk_edges(gpu_lib, n, F):
    import torch
    rng = np.random.default_rng(n + F)
    pos = rng.random((n, 3)).astype(np.float32)
    vals = rng.normal(size=(F, n)).astype(np.float32)
    if n > 100:
        pos[::97, 1] = 1.5          # outside
        pos[5, 2] = np.nan
        vals[0, 7] = np.inf
        vals[F - 1, 11] = np.nan
        vals[:, 13] = 0.0
    _check(gpu_lib, torch, (17, 13, 11), pos, vals, f"ordered deposit n={n} F={F}")


@pytest.mark.parametrize("order", ["sorted", "one cell", "two ends"])
@pytest.mark.parametrize("F", [1, 4])
def test_long_and_empty_runs(gpu_lib, order, F):
    """Particles sorted by cell (a chunk is few long runs, most runs of a
    tile empty), all in one cell, and in two far cells by turns."""
    import torch
    shape, n = (64, 64, 64), 150_000
    rng = np.random.default_rng(3)
    pos = rng.random((n, 3)).astype(np.float32)
    if order == "sorted":
        pos = pos[np.lexsort((pos[:, 0], (pos[:, 1] * 64).astype(int), (pos[:, 2] * 64).astype(int)))]
    elif order == "one cell":
        pos = (np.float32(0.5) + pos * np.float32(1 / 128))
    else:
        pos = pos * np.float32(1 / 128)
        pos[1::2] += np.float32(0.99)
    vals = rng.normal(size=(F, n)).astype(np.float32)
    _check(gpu_lib, torch, shape, np.ascontiguousarray(pos), vals, f"ordered deposit {order} F={F}")


def test_more_chunks_than_runs_summed_at_once(gpu_lib):
    """635 chunks of 2048 on 768 tiles: more runs per tile than a quarter
    workgroup numbers at once (512)."""
    import torch
    shape, n = (256, 256, 192), 1_300_000
    p = inputs.uniform_bed(inputs.HexBox((0, 0, 0), (1, 1, 1), shape), n, 1, seed=4)
    _check(gpu_lib, torch, shape, p.pos, p.values, "ordered deposit 635 chunks")


@pytest.mark.parametrize("scale", [1e-38, 1e-30, 1e30])
def test_finished_values_at_the_ends_of_float32(gpu_lib, scale):
    """Fields near float32's smallest and largest normal numbers: the finished
    value is the rounded quotient there too (denormal results included)."""
    import torch
    rng = np.random.default_rng(8)
    n = 30_000
    pos = rng.random((n, 3)).astype(np.float32)
    vals = (rng.normal(size=(2, n)) * scale).astype(np.float32)
    _check(gpu_lib, torch, (32, 16, 8), pos, vals, f"ordered deposit values of {scale}")


@pytest.mark.parametrize("switch", ["CGD_DEPOSIT_NSUB", "CGD_DEPOSIT_BIN_NSUB"])
def test_switches_of_the_counting_passes_reach_them(gpu_lib, switch, monkeypatch):
    """Either switch alone: counted, scattered (timing kind "deposit_scatter"), the same bits."""
    import torch
    rng = np.random.default_rng(5)
    pos = rng.random((50_000, 3)).astype(np.float32)
    vals = rng.normal(size=(2, 50_000)).astype(np.float32)
    monkeypatch.setenv(switch, "2")
    _check(gpu_lib, torch, (40, 30, 20), pos, vals, f"deposit {switch}")
    mesh = gpu_lib.HexMesh((40, 30, 20))
    gpu_lib.timing_enable(mesh, True)
    gpu_lib.deposit(mesh, torch.from_numpy(pos).cuda(), torch.from_numpy(vals).cuda(), stats=True)
    gpu_lib.diffuse(mesh, torch.ones((1, mesh.cells), device="cuda"), 0.05, 1)
    assert gpu_lib.timing_read(mesh)["deposit_scatter"][0] == 1


# Full-size chunks (16384 particles at one field, 8192 at two and three, 6144 at four), which start at 80 chunks: one
# particle short of the line, at it, and a ragged rest; more than 2048 records per tile of 8192 sums and more, for the
# 1024-thread accumulation
@pytest.mark.parametrize("F,n", [(1, 80 * 16384 - 1), (1, 80 * 16384), (2, 80 * 8192 - 1), (2, 80 * 8192 + 4321),
                                 (3, 80 * 8192), (4, 80 * 6144 - 1), (4, 80 * 6144), (2, 256 * 8192 + 4321),
                                 (3, 256 * 8192 + 7), (4, 256 * 6144 + 6143)])
def test_full_size_chunks(gpu_lib, F, n):
    import torch
    rng = np.random.default_rng(F)
    pos = rng.random((n, 3)).astype(np.float32)
    vals = rng.normal(size=(F, n)).astype(np.float32)
    pos[::1001, 1] = 1.5            # outside
    pos[5, 2] = np.nan
    vals[0, 7] = np.inf
    vals[F - 1, n - 1] = np.nan
    shape = (128, 128, 65) if F == 4 else (128, 128, 130)
    _check(gpu_lib, torch, shape, pos, vals, f"ordered deposit, full chunks F={F} n={n}")


# rectilinear grids: full-size chunks from 200 to 256 and from 400 on
@pytest.mark.parametrize("F,n", [(1, 200 * 16384 - 1), (1, 200 * 16384 + 9), (2, 256 * 8192 + 55), (2, 257 * 8192),
                                 (3, 399 * 8192), (4, 400 * 6144 + 1)])
def test_full_size_chunks_rectilinear(gpu_lib, F, n):
    import torch
    cgd = gpu_lib
    shape = (128, 128, 65 if F == 4 else 130)
    rng = np.random.default_rng(F)
    edges = []
    for m in shape:
        w = 0.4 + rng.random(m)
        e = np.concatenate([[0.0], np.cumsum(w)]) / w.sum()
        e[-1] = 1.0
        edges.append(e)
    pos = (1.02 * rng.random((n, 3)) - 0.01).astype(np.float32)
    vals = rng.normal(size=(F, n)).astype(np.float32)
    print(f"case: ordered deposit, full chunks, rectilinear F={F}", flush=True)
    mesh = cgd.RectMesh(*edges)
    acc = torch.empty((F, mesh.cells), dtype=torch.int64, device="cuda")
    field, st = cgd.deposit(mesh, torch.from_numpy(pos).cuda(), torch.from_numpy(vals).cuda(), acc=acc, stats=True)
    ref = O.deposit_rect(pos, vals, edges)
    assert np.array_equal(acc.cpu().numpy(), ref["acc"])
    assert np.array_equal(field.cpu().numpy().view(np.uint32), ref["field32"].view(np.uint32))
    assert st.n_dropped == ref["n_dropped"]


@pytest.mark.parametrize("F", [2, 4])
def test_full_size_chunks_batched(gpu_lib, F):
    """Uneven snapshots (one empty, one of one particle) whose total takes
    full-size chunks: each the bits of its own call, which takes small ones."""
    import torch
    cgd = gpu_lib
    shape = (128, 128, 40)
    counts = [900_001, 0, 1, 700_000, 600_123]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(off[-1])
    assert n >= 256 * 8192
    rng = np.random.default_rng(F)
    pos = torch.from_numpy(rng.random((n, 3)).astype(np.float32)).cuda()
    vals = torch.from_numpy(rng.normal(size=(F, n)).astype(np.float32)).cuda()
    mesh = cgd.HexMesh(shape)
    print(f"case: ordered deposit, full chunks, batched F={F}", flush=True)
    out = cgd.coarse_grain_batched(mesh, off, pos, vals, 0.05, 2)
    for j in range(len(counts)):
        s = slice(int(off[j]), int(off[j + 1]))
        one = cgd.coarse_grain(mesh, pos[s].contiguous(), vals[:, s].contiguous(), 0.05, 2)[0]
        assert torch.equal(one.view(torch.int32), out[j].view(torch.int32)), j


def test_sparse_grid_of_largest_tiles(gpu_lib):
    """One particle in a thousand cells, tiles of 16384 sums, a ragged one: a
    whole workgroup per tile; and the same cells with more records per tile
    than a quarter workgroup takes, in smaller tiles (1024 cells each)."""
    import torch
    rng = np.random.default_rng(6)
    for shape, n in (((256, 256, 130), 9_000), ((128, 64, 64), 512 * 16384 + 3)):
        pos = rng.random((n, 3)).astype(np.float32)
        vals = rng.normal(size=(1, n)).astype(np.float32)
        _check(gpu_lib, torch, shape, pos, vals, f"ordered deposit {shape} n={n}")
