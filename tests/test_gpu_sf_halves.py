"""Structure factors of lists whose mates are not mates, on both sides of the rules that split the
launch: the halves of the list in blocks of their own (up to 1024 blocks) or one after the other, and
chunks by floor or by ceil (410 blocks of reflections).  Against the sum in binary64, 5e-6 of the sum
of the amplitudes as derived in test_gpu_sf_mates; a list with one broken pair runs the pairs of one
block alone, and the others' mates stay conjugates bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import atoms_to_device  # noqa: E402
from paper_2608_23245_amd import binding as B  # noqa: E402
from test_gpu_sf_mates import exact, lists  # noqa: E402


@pytest.mark.parametrize("kind", ["one", "none"])
@pytest.mark.parametrize("n,n_atoms", [(8192, 4095), (8192, 4160), (8193, 4096), (209409, 130), (209923, 130), (2, 130000)])
def test_halves(n, n_atoms, kind):
    wl = W.config0()
    rng = np.random.default_rng(n + n_atoms)
    atoms = atoms_to_device(wl.atoms)
    n_types = atoms["ff"].shape[0]
    f32 = lambda lo, hi: torch.as_tensor(rng.uniform(lo, hi, n_atoms), dtype=torch.float32).cuda()  # noqa: E731
    atoms.update({k: f32(-0.3, 1.3) for k in "xyz"}, B=f32(2, 15), occ=f32(0.2, 1.0),
                 type=torch.as_tensor(rng.integers(0, n_types, n_atoms), dtype=torch.int32).cuda())
    hkl = torch.as_tensor(lists(n, kind, n), dtype=torch.int32).cuda()
    cell = B.make_cell(wl.cell)
    print(f"{n} reflections ({kind}), {n_atoms} atoms", flush=True)
    F, F2 = B.structure_factors(cell, atoms, hkl)
    got = torch.complex(F.reshape(-1, 2)[:, 0].double(), F.reshape(-1, 2)[:, 1].double())
    want, size = exact(cell, atoms, hkl)
    assert bool(((got - want).abs() <= 5e-6 * size).all())
    assert bool(((F2.double() - want.abs() ** 2).abs() <= 2 * 5e-6 * size * size).all())
    if kind == "one" and n > 1024:
        own = (hkl.flip(0) != -hkl).any(1)  # the broken pair
        assert int(own.sum()) == 2
        same = got.flip(0).conj().resolve_conj() == got
        block = torch.arange(n, device="cuda")
        block = torch.minimum(block, n - 1 - block) // 512
        assert bool(same[block != block[own][0]].all())
