"""The splat where a wave's lanes walk their own nodes (patches wide against the support): one
patch and its remainders, one row of nodes, windows below and above what is kept in LDS, each
lineshape, sharp and broad supports.  Against the binary64 model with the bounds of the splat's own
test (relative L2 1e-4, per pixel 1e-3 above a thousandth of the maximum), and the number of
(sample, node) terms equal up to float32 rounding at the edge of the support: a window that
missed a node would show there."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("lineshape", [0, 1, 2])
@pytest.mark.parametrize("n_s,nodes,sharper", [(1, 16, 1.0), (7, 12, 3.0), (8, 16, 3.0), (9, 17, 3.0), (16, 24, 4.0),
                                               (16, 40, 4.0), (24, 20, 1.0), (33, 9, 6.0)])
def test_lanes_vs_oracle(n_s, nodes, sharper, lineshape):
    wl = W.small(60 + n_s, width=30, height=26, sigma_theta=0.05, gamma_theta=0.02, n_nodes=nodes, lineshape=lineshape,
                 g=(0.02, 0.01, 0.0))
    wl = dataclasses.replace(wl, dis=dataclasses.replace(wl.dis, N_base=tuple(sharper * v for v in wl.dis.N_base)))
    hkl = O.enumerate_hkl(wl.cell, wl.quad.d_min, wl.quad.d_max)
    hkl = np.ascontiguousarray(hkl[~O.extinct_mask(hkl, wl.dis, wl.quad.extinction)])[:200]
    print(f"n_s {n_s}, {nodes} nodes, {hkl.shape[0]} reflections", flush=True)
    model = B.make_model(wl)
    h = torch.from_numpy(np.ascontiguousarray(hkl, dtype=np.int32)).cuda()
    F = O.structure_factors_c(hkl, wl.cell, wl.atoms)
    F2 = torch.as_tensor((F.real ** 2 + F.imag ** 2).astype(np.float32)).cuda()
    refl, _ = B.reflection_prep(model, h, F2)
    table = B.node_table(model)
    n_r = 6
    img = B.splat(model, h, refl, table, n_r, n_s).cpu().numpy().astype(np.float64)
    cnt = B.splat(model, h, refl, table, n_r, n_s, count=True)
    ref, n_ref = O.splat(wl, O.prepare(wl, hkl=hkl, F=F, cull_extinct=False), n_r, n_s, count=True)
    assert abs(cnt - n_ref) <= 1e-5 * n_ref + 2
    if ref.max() > 0:
        assert np.linalg.norm(img - ref) <= 1e-4 * np.linalg.norm(ref)
        big = ref > 1e-3 * ref.max()
        assert np.max(np.abs(img[big] - ref[big]) / ref[big]) <= 1e-3
