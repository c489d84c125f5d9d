"""Work units of the balanced launches at the counts where a wave's way of taking them changes:
one unit, one wave's width, and the number of waves of a launch (4 to 8 per SIMD of 256 compute
units) with one more and one less.  The lists are those of a crop of the medium model cut to
the wanted number of pairs, one pair per unit; the image is the per-tile launch's over the same
lists, whose terms are the same and only grouped otherwise (2e-6 of the largest value, the
tolerance of the balanced launch's own test), and the adjoint's sums are the per-tile ones to
the rounding of binary64 atomic adds."""
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
    wl = dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, width=128, height=128, center_x=64.0, center_y=64.0,
                                                          tile_w=16, unit_pairs=1))
    model = B.make_model(wl)
    hkl = B.enumerate_hkl(model.cell, wl.quad.d_min, wl.quad.d_max, extinction=(0.03, 0.03, 0.0, 30.0))
    _, F2 = B.structure_factors(model.cell, atoms_to_device(wl.atoms), hkl, want_F=False)
    refl, cull = B.reflection_prep(model, hkl, F2)
    nodes = B.node_table(model)
    pix, tile = B.pixel_map(model.geom)
    off, idx = B.cull(model.geom, tile, cull)
    return model, refl, nodes, pix, tile, off.cpu().numpy(), idx.cpu().numpy()


def cut(off, idx, total):
    """total of the lists' pairs, spread evenly over them, as lists of the same tiles."""
    pick = np.linspace(0, idx.shape[0] - 1, total).astype(np.int64)
    assert np.unique(pick).shape[0] == total
    tile_of = np.searchsorted(off, pick, side="right") - 1
    o = np.concatenate([[0], np.cumsum(np.bincount(tile_of, minlength=off.shape[0] - 1))])
    return torch.as_tensor(o, dtype=torch.int64).cuda(), torch.as_tensor(idx[pick], dtype=torch.int32).cuda()


@pytest.mark.parametrize("total", [1, 64, 65] + [1024 * w + d for w in range(4, 9) for d in (-1, 0, 1)])
def test_units_around_the_number_of_waves(crop, total):
    model, refl, nodes, pix, tile, off, idx = crop
    o, i = cut(off, idx, total)
    print(f"{total} units", flush=True)
    G = torch.as_tensor(np.random.default_rng(3).normal(size=(128, 128)), dtype=torch.float32).cuda()
    ws = B.balanced_workspace(model, total)
    img = B.profile_balanced(model, refl, nodes, pix, tile, o, i, ws=ws)
    ref = B.profile(model, refl, nodes, pix, tile, o, i)
    sums = B.profile_adjoint_balanced(model, refl, nodes, pix, tile, o, i, G, ws)
    want = B.profile_adjoint(model, refl, nodes, pix, tile, o, i, G)
    scale = ref.abs().max().item()
    assert (img - ref).abs().max().item() <= 2e-6 * scale
    s = want.abs().amax(dim=0).clamp(min=1e-300)
    assert ((sums - want).abs() / s).max().item() <= 1e-10
