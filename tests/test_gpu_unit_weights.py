"""Units cut by the weight of their pairs (the balanced launches' own choice, for lists short
against the node grid) at one pair, and on both sides of the pair counts between which they are
weighed (8192, and 2048 times the nodes), on lists cut evenly from a crop of the
medium model, whose pairs have from none to every node in their window.  The image is the
per-tile launch's over the same lists up to the grouping of its sums (2e-6 of the largest value,
the tolerance of the balanced launch's own test), with and without a launch order bit for bit,
and the adjoint over the same units has the per-tile sums to the rounding of binary64 adds."""
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


@pytest.fixture(scope="module")
def crop():
    wl = W.config1()
    wl = dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, width=200, height=184, center_x=100.0, center_y=92.0,
                                                          tile_w=16))
    model = B.make_model(wl)
    hkl = B.enumerate_hkl(model.cell, wl.quad.d_min, wl.quad.d_max, extinction=(0.03, 0.03, 0.0, 30.0))
    _, F2 = B.structure_factors(model.cell, atoms_to_device(wl.atoms), hkl, want_F=False)
    refl, cull = B.reflection_prep(model, hkl, F2)
    pix, tile = B.pixel_map(model.geom)
    off, idx = B.cull(model.geom, tile, cull)
    return wl, hkl, F2, pix, tile, off.cpu().numpy(), idx.cpu().numpy()


@pytest.mark.parametrize("lineshape", [0, 1, 2])
@pytest.mark.parametrize("nodes,total", [(16, 1), (16, 63), (16, 8192), (24, 8193), (64, 20000), (2, 8192), (2, 8193), (5, 51200),
                                         (5, 51201)])
def test_weighed_units(crop, nodes, total, lineshape):
    wl, hkl, F2, pix, tile, off, idx = crop
    wl = dataclasses.replace(wl, quad=dataclasses.replace(wl.quad, n_nodes=nodes),
                             dis=dataclasses.replace(wl.dis, lineshape=lineshape))
    model = B.make_model(wl)
    refl, _ = B.reflection_prep(model, hkl, F2)
    table = B.node_table(model)
    pick = np.linspace(0, idx.shape[0] - 1, total).astype(np.int64)
    assert np.unique(pick).shape[0] == total
    tile_of = np.searchsorted(off, pick, side="right") - 1
    o = torch.as_tensor(np.concatenate([[0], np.cumsum(np.bincount(tile_of, minlength=off.shape[0] - 1))])).cuda()
    i = torch.as_tensor(idx[pick], dtype=torch.int32).cuda()
    order = B.tile_order(model.geom, o)
    print(f"{total} pairs, {nodes} nodes, {'by weight' if 8192 < total <= 2048 * nodes * nodes else 'by number'}", flush=True)
    G = torch.as_tensor(np.random.default_rng(4).normal(size=(184, 200)), dtype=torch.float32).cuda()
    ref = B.profile(model, refl, table, pix, tile, o, i)
    want = B.profile_adjoint(model, refl, table, pix, tile, o, i, G)
    ws = B.balanced_workspace(model, total)
    plain = B.profile_balanced(model, refl, table, pix, tile, o, i, ws=ws)
    img = B.profile_balanced(model, refl, table, pix, tile, o, i, order=order, ws=ws)
    sums = B.profile_adjoint_balanced(model, refl, table, pix, tile, o, i, G, ws, order=order)
    scale = ref.abs().max().item()
    assert (img - ref).abs().max().item() <= 2e-6 * scale
    assert torch.equal(img, plain)
    assert (sums - want).abs().max().item() <= 1e-9 * want.abs().max().item()
