"""Structure factors with a row of the form-factor table that no atom uses and that holds no
numbers (a table built for more elements than a model has): the row has no part in any sum, so
F is finite and has the bits it has with a row of numbers there, at atom counts that fill a
group of eight, a chunk or a block and counts that do not."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import atoms_to_device  # noqa: E402
from paper_2608_23245_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("unused", [0, 1, 2])
@pytest.mark.parametrize("n,n_atoms", [(5, 1), (6, 7), (300, 8), (301, 257), (40, 2051), (140000, 4099)])
def test_unused_row(n, n_atoms, unused, value):
    wl = W.config0()
    rng = np.random.default_rng(n + n_atoms)
    atoms = atoms_to_device(wl.atoms)
    f32 = lambda lo, hi: torch.as_tensor(rng.uniform(lo, hi, n_atoms), dtype=torch.float32).cuda()  # noqa: E731
    used = [t for t in range(3) if t != unused]
    atoms.update({k: f32(-0.3, 1.3) for k in "xyz"}, B=f32(2, 15), occ=f32(0.2, 1.0),
                 type=torch.as_tensor(rng.choice(used, n_atoms), dtype=torch.int32).cuda())
    cell = B.make_cell(wl.cell)
    h = rng.integers(-20, 21, size=(n // 2, 3))
    h = np.concatenate([h, np.zeros((n % 2, 3), dtype=h.dtype), -h[::-1]])
    for hkl in (torch.as_tensor(h, dtype=torch.int32).cuda(), torch.as_tensor(np.abs(h), dtype=torch.int32).cuda()):
        F0, F20 = B.structure_factors(cell, atoms, hkl)
        ff = atoms["ff"].clone()
        ff.view(-1, 9)[unused] = value
        F, F2 = B.structure_factors(cell, dict(atoms, ff=ff), hkl)
        print(f"{n} reflections, {n_atoms} atoms, row {unused} {value}", flush=True)
        assert bool(torch.isfinite(F).all()) and F.abs().max() > 0
        assert torch.equal(F, F0) and torch.equal(F2, F20)
