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
