"""Launches of more threads than one grid dimension holds.  HIP refuses 2^32 threads along one
dimension and of more runs the excess alone, without an error.

The balanced pattern launch of a detector of 2^24 tiles and more (its unit sums take four waves
a tile): short lists in tiles spread over it and in its last ones, against the per-tile launch over
the same lists (float32 rounding of the same sums, 1e-5 of relative L2) and exactly zero in every
tile without a list.  The pair reduction of 2^28 reflections and more (sixteen lanes each): rows
spread over the list and in its last places, whole numbers that any order sums exactly."""
import ctypes
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import atoms_to_device  # noqa: E402
from paper_2608_23245_amd import binding as B  # noqa: E402


@pytest.fixture(autouse=True)
def give_memory_back():
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("columns", [4096, 4097])
def test_balanced_launch_of_many_tiles(columns):
    wl = W.small(91, width=8 * columns, height=8 * 4096, d_min=5.0)
    wl = dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, pixel=0.8 * 24 / (8 * columns), tile_waves=2))
    model = B.make_model(wl)
    hkl = B.enumerate_hkl(model.cell, wl.quad.d_min, wl.quad.d_max)
    _, F2 = B.structure_factors(model.cell, atoms_to_device(wl.atoms), hkl, want_F=False)
    refl, _ = B.reflection_prep(model, hkl, F2)
    nodes = B.node_table(model)
    pix, tile = B.pixel_map(model.geom)
    n_tiles, n = 4096 * columns, int(hkl.shape[0])
    rng = np.random.default_rng(columns)
    listed = np.concatenate([rng.choice(n_tiles - 8, 300, replace=False), np.arange(n_tiles - 8, n_tiles)])
    per = torch.zeros(n_tiles + 1, dtype=torch.int64, device="cuda")
    per[torch.as_tensor(listed).cuda() + 1] = n
    off = per.cumsum(0)
    idx = torch.arange(n, dtype=torch.int32, device="cuda").repeat(len(listed))
    p = B._ptr
    cap = int(idx.shape[0])
    ws = B.balanced_workspace(model, cap)
    img = torch.full((wl.geom.height, wl.geom.width), -1.0, device="cuda")
    print(f"{n_tiles} tiles, {cap} pairs", flush=True)
    B._check(B.lib().fdtbx_profile_balanced(ctypes.byref(model), p(refl), p(nodes), p(pix), p(tile), p(off), p(idx), None, cap,
                                            p(img), p(ws), int(ws.numel()), B._stream()))
    ref = B.profile(model, refl, nodes, pix, tile, off, idx)
    torch.cuda.synchronize()
    in_list = torch.zeros(n_tiles, dtype=torch.bool, device="cuda")
    in_list[torch.as_tensor(listed).cuda()] = True
    tiles = img.view(4096, 8, columns, 8).permute(0, 2, 1, 3).reshape(n_tiles, 64)
    assert torch.count_nonzero(tiles[~in_list]).item() == 0
    ref = ref.view(4096, 8, columns, 8).permute(0, 2, 1, 3).reshape(n_tiles, 64)[in_list].double()
    assert ref.max() > 0
    assert ((tiles[in_list].double() - ref).norm() / ref.norm()).item() <= 1e-5


@pytest.mark.parametrize("n", [1 << 28, (1 << 28) + 1])
def test_pair_reduction_of_many_reflections(n):
    rng = np.random.default_rng(n)
    rows = torch.as_tensor(np.unique(np.concatenate([rng.integers(0, n, 200), np.arange(n - 3, n)]))).cuda()
    length = torch.as_tensor(rng.integers(1, 40, rows.shape[0])).cuda()
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    ptr[rows + 1] = length
    ptr = ptr.cumsum_(0)
    total = int(length.sum())
    part = torch.as_tensor(rng.integers(-99, 100, (total, 12)), dtype=torch.float32).cuda()
    pairs = torch.as_tensor(rng.permutation(total), dtype=torch.int32).cuda()
    print(f"{n} reflections, {total} pairs", flush=True)
    sums = torch.full((n, 6), -1.0, dtype=torch.float64, device="cuda")
    p = B._ptr
    B._check(B.lib().fdtbx_pair_reduce(n, p(ptr), p(pairs), p(part), None, 0, p(sums), B._stream()))
    torch.cuda.synchronize()
    at = 0
    for r, m in zip(rows.tolist(), length.tolist()):
        assert torch.equal(sums[r], part[pairs[at:at + m].long(), :6].double().sum(0)), r
        at += m
    sums[rows] = 0.0
    assert torch.count_nonzero(sums).item() == 0


def test_clearing_of_many_partials():
    """Per-pair sums of 2^32 values and more (358 million pairs of capacity): cleared to the last."""
    wl = W.small(93)
    model = B.make_model(wl)
    hkl = B.enumerate_hkl(model.cell, wl.quad.d_min, wl.quad.d_max)
    _, F2 = B.structure_factors(model.cell, atoms_to_device(wl.atoms), hkl, want_F=False)
    refl, cull = B.reflection_prep(model, hkl, F2)
    pix, tile = B.pixel_map(model.geom)
    off, idx = B.cull(model.geom, tile, cull)
    cap = (1 << 32) // 12 + 1
    part = torch.full((cap, 12), -1.0, device="cuda")
    G = torch.zeros((wl.geom.height, wl.geom.width), device="cuda")
    p = B._ptr
    print(f"{cap} pairs of capacity, {idx.numel()} listed", flush=True)
    B._check(B.lib().fdtbx_profile_adjoint_pairs(ctypes.byref(model), p(refl), p(B.node_table(model)), p(pix), p(tile), p(off), p(idx),
                                                 None, int(hkl.shape[0]), cap, p(G), p(part), B._stream()))
    torch.cuda.synchronize()
    assert torch.count_nonzero(part).item() == 0
