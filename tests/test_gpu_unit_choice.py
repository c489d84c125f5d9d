"""unit_pairs 0 against the same launch with unit_pairs = fdtbx_unit_pairs(n_pairs), at the pair counts
between which the library's own choice weighs the pairs: the same bits up to 8192 pairs and above 2048
times the nodes, where both cut by number, and between the two the same sums in other groups (2e-6 of
the largest value, the tolerance of the balanced launch's own test)."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import binding as B  # noqa: E402
from test_gpu_unit_weights import crop  # noqa: E402,F401


@pytest.mark.parametrize("nodes,total,same", [(16, 40, True), (16, 8192, True), (24, 8193, False), (5, 51200, False),
                                              (5, 51201, True)])
def test_zero_against_the_stated_size(crop, nodes, total, same):  # noqa: F811
    wl, hkl, F2, pix, tile, off, idx = crop
    wl = dataclasses.replace(wl, quad=dataclasses.replace(wl.quad, n_nodes=nodes))
    pick = np.linspace(0, idx.shape[0] - 1, total).astype(np.int64)
    tile_of = np.searchsorted(off, pick, side="right") - 1
    o = torch.as_tensor(np.concatenate([[0], np.cumsum(np.bincount(tile_of, minlength=off.shape[0] - 1))])).cuda()
    i = torch.as_tensor(idx[pick], dtype=torch.int32).cuda()
    img = []
    for u in (0, B.unit_pairs(total)):
        model = B.make_model(dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, unit_pairs=u)))
        refl, _ = B.reflection_prep(model, hkl, F2)
        img.append(B.profile_balanced(model, refl, B.node_table(model), pix, tile, o, i))
    print(f"{total} pairs, {nodes} nodes, {u} pairs a unit", flush=True)
    assert img[1].max() > 0
    assert torch.equal(*img) if same else (img[0] - img[1]).abs().max().item() <= 2e-6 * img[1].max().item()
