"""Structure factors of lists that are symmetric, in part or not at all, at the sizes where the
kernel's split changes: one reflection, the middle of an odd list, one block's reflections (256
or 512 of the first half) and the atoms of a chunk (64) and of a group (8).  Against the sum in binary64;
a term carries the float32 rounding of its phase (1.9e-7 of its size), of its exponent and
amplitude (under 2e-6 for exponents up to 10), and a group's float32 sum of eight terms adds
6e-8 a step: 5e-6 of the sum of the amplitudes in all.  The mate of every
reflection in a symmetric list is its conjugate."""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import atoms_to_device  # noqa: E402
from paper_2608_23245_amd import binding as B  # noqa: E402


def exact(cell, atoms, hkl):
    """F and the sum of |amplitude|, binary64."""
    h = hkl.double()
    ca, cb, cg, sa = math.cos(cell.alpha), math.cos(cell.beta), math.cos(cell.gamma), math.sin(cell.alpha)
    ay, az = cell.a * (cg - ca * cb) / sa, cell.a * cb
    A = np.array([[math.sqrt(cell.a ** 2 - ay ** 2 - az ** 2), ay, az], [0, cell.b * sa, cell.b * ca], [0, 0, cell.c]])
    q = h @ torch.as_tensor(np.linalg.inv(A).T, device=h.device)
    s2 = 0.25 * (q * q).sum(1)
    ff = atoms["ff"].double().reshape(-1, 9)
    f = ff[None, :, 8] + (ff[None, :, :4] * torch.exp(-ff[None, :, 4:8] * s2[:, None, None])).sum(2)
    F = torch.zeros(h.shape[0], dtype=torch.complex128, device=h.device)
    size = torch.zeros(h.shape[0], dtype=torch.float64, device=h.device)
    for j in range(0, atoms["x"].shape[0], 256):
        s = slice(j, j + 256)
        amp = atoms["occ"][s].double() * f[:, atoms["type"][s].long()] * torch.exp(-atoms["B"][s].double() * s2[:, None])
        ph = h @ torch.stack([atoms["x"][s], atoms["y"][s], atoms["z"][s]]).double()
        F += (amp * torch.exp(2j * math.pi * (ph - ph.floor()))).sum(1)
        size += amp.abs().sum(1)
    return F, size


def lists(n, kind, seed):
    """n reflections: "symmetric" has mate n - 1 - i for every i (an odd list the origin in its
    middle), "one" breaks a single one of them, "none" is a random list."""
    rng = np.random.default_rng(seed)
    if kind == "none":
        return rng.integers(-40, 41, size=(n, 3))
    h = rng.integers(-40, 41, size=(n // 2, 3))
    h = np.concatenate([h, np.zeros((n % 2, 3), dtype=h.dtype), -h[::-1]])
    if kind == "one":
        h[n - 1 - min(300, n // 4)] += (0, 0, 1)
    return h


@pytest.mark.parametrize("kind", ["symmetric", "one", "none"])
@pytest.mark.parametrize("n,n_atoms", [(1, 1), (2, 63), (3, 64), (255, 65), (512, 257), (513, 2049), (1023, 300), (1024, 5000),
                                       (1025, 64), (2051, 700), (70001, 4300)])
def test_mates_and_splits(n, n_atoms, kind):
    wl = W.config0()
    rng = np.random.default_rng(n + n_atoms)
    atoms = atoms_to_device(wl.atoms)
    n_types = atoms["ff"].shape[0]
    f32 = lambda lo, hi: torch.as_tensor(rng.uniform(lo, hi, n_atoms), dtype=torch.float32).cuda()  # noqa: E731
    atoms.update({k: f32(-0.3, 1.3) for k in "xyz"}, B=f32(2, 15), occ=f32(0.2, 1.0),
                 type=torch.as_tensor(rng.integers(0, n_types, n_atoms), dtype=torch.int32).cuda())
    cell = B.make_cell(wl.cell)
    hkl = torch.as_tensor(lists(n, kind, n), dtype=torch.int32).cuda()
    print(f"{n} reflections ({kind}), {n_atoms} atoms", flush=True)
    F, F2 = B.structure_factors(cell, atoms, hkl)
    got = torch.complex(F.reshape(-1, 2)[:, 0].double(), F.reshape(-1, 2)[:, 1].double())
    want, size = exact(cell, atoms, hkl)
    assert bool(((got - want).abs() <= 5e-6 * size).all())
    assert bool(((F2.double() - want.abs() ** 2).abs() <= 2 * 5e-6 * size * size).all())
    if kind == "symmetric":
        assert torch.equal(got.flip(0).conj().resolve_conj()[:n // 2], got[:n // 2])
