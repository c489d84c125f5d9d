"""The cylindrical average with several workgroups per tile (fdtbx_profile_cyl_split) against one
per tile (fdtbx_profile_cyl) over the same lists, cut to the lengths where the sharing changes:
no pair, one, one less and one more than the workgroups of a tile, and so on.  Both evaluate the
same (pixel, ring point, node) terms, all positive; they group the float32 sums differently
and start the binary64 rotation of the ring at other points, which moves a coordinate by at
most its last float32 bit.  1e-5 of relative L2 is a tenth of the bound that either keeps against
the binary64 model.  A folded detector takes the unfolded one's workgroups per tile."""
import ctypes
import dataclasses

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import atoms_to_device  # noqa: E402
from paper_2608_23245_amd import binding as B  # noqa: E402


@pytest.fixture(scope="module")
def lists():
    wl = W.config1()
    wl = dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, width=128, height=128, center_x=64.0, center_y=64.0,
                                                          tile_w=16))
    model = B.make_model(wl)
    hkl = B.enumerate_hkl(model.cell, wl.quad.d_min, wl.quad.d_max, extinction=(0.03, 0.03, 0.0, 30.0))
    _, F2 = B.structure_factors(model.cell, atoms_to_device(wl.atoms), hkl, want_F=False)
    pix, tile = B.pixel_map(model.geom)
    off, idx = B.cull(model.geom, tile, B.cyl_records(model, hkl))
    return wl, hkl, F2, pix, off.cpu(), idx.cpu()


def cut(off, idx, n):
    """n[t % len(n)] pairs of each tile's list, spread evenly over it (all of a shorter list)."""
    rows = []
    for t in range(off.shape[0] - 1):
        row = idx[off[t]:off[t + 1]]
        m = min(row.shape[0], n[t % len(n)])
        rows.append(row[((2 * torch.arange(m) + 1) * row.shape[0]) // (2 * max(m, 1))])
    o = torch.tensor([0] + [r.shape[0] for r in rows], dtype=torch.int64).cumsum(0)
    return o.cuda(), torch.cat(rows + [torch.zeros(1, dtype=torch.int32)]).cuda()


@pytest.mark.parametrize("lineshape", [0, 1, 2])
@pytest.mark.parametrize("waves,n", [(0, (0, 1, 2, 3)), (1, (1, 31, 33, 62)), (2, (63, 64, 65, 5)), (4, (0, 127, 128, 129))])
def test_split_against_one_workgroup_per_tile(lists, waves, n, lineshape):
    wl, hkl, F2, pix, off, idx = lists
    wl = dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, tile_waves=waves),
                             dis=dataclasses.replace(wl.dis, lineshape=lineshape))
    model = B.make_model(wl)
    refl, _ = B.reflection_prep(model, hkl, F2)
    tiles = off.shape[0] - 1
    nbytes = B.lib().fdtbx_cyl_workspace(ctypes.byref(model.geom))
    print(f"tiles {tiles}, {nbytes // (256 * tiles)} workgroups each, tile_waves {waves}, lists of {n}", flush=True)
    assert nbytes == 64 * 256 * tiles  # 256 tiles: 64 workgroups each
    o, i = cut(off, idx, n)
    nodes = B.node_table(model)
    arc = 2e-3
    got = B.profile_cyl(model, refl, nodes, pix, o, i, arc)
    ref = torch.empty_like(got)
    p = B._ptr
    call = (ctypes.byref(model), p(refl), p(nodes), p(pix), p(o), p(i), None, arc)
    B._check(B.lib().fdtbx_profile_cyl(*call, p(ref), None, B._stream()))
    assert ref.max() > 0
    assert ((got - ref).double().norm() / ref.double().norm()).item() <= 1e-5
    order = B.tile_order(model.geom, o)
    assert torch.equal(B.profile_cyl(model, refl, nodes, pix, o, i, arc, order=order), got)


def test_split_workspace_is_checked(lists):
    wl, hkl, F2, pix, off, idx = lists
    model = B.make_model(wl)
    refl, _ = B.reflection_prep(model, hkl, F2)
    p = B._ptr
    o, i = cut(off, idx, (1,))
    img = torch.full((128, 128), -1.0, device="cuda")
    need = B.lib().fdtbx_cyl_workspace(ctypes.byref(model.geom))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    call = (ctypes.byref(model), p(refl), p(B.node_table(model)), p(pix), p(o), p(i), None, 2e-3, p(img))
    short = B.lib().fdtbx_profile_cyl_split(*call, p(ws), need - 1, B._stream())
    none = B.lib().fdtbx_profile_cyl_split(*call, None, need, B._stream())
    torch.cuda.synchronize()
    assert short != 0 and none != 0 and bool((img == -1.0).all())
    big = W.config1()
    big = B.make_model(dataclasses.replace(big, geom=dataclasses.replace(big.geom, width=1024, height=1024)))
    assert B.lib().fdtbx_cyl_workspace(ctypes.byref(big.geom)) == 0
