"""The fixed-order sums of the adjoint by either route: pairs found by searching the tiles' lists
(few reflections times tiles) and pairs sorted by reflection.  The searched sums are compared
with the sorted route over the same partials of the same pass at one tile, at ragged ones, at
each fold and on both sides of the rule; both add the same float32 partials in binary64, so
their gradients agree to the last float32 place of a group's largest value.  The reduction
itself is compared with numpy at the row lengths around its sixteen lanes, to 1e-13 of the sum
of magnitudes (binary64 sums of at most 1000 terms)."""
import ctypes
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import autograd as AG  # noqa: E402
from paper_2608_23245_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("lengths", [[0], [1, 0, 15, 16, 17, 31, 33], [1000] + [2] * 40])
@pytest.mark.parametrize("mates", ["none", "updown", "given"])
def test_pair_reduce_row_lengths(lengths, mates):
    rng = np.random.default_rng(len(lengths))
    n, total = len(lengths), sum(lengths)
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    pairs = rng.permutation(total)
    part = rng.normal(size=(total, 12)).astype(np.float32)
    mate = rng.integers(-1, n, size=n)
    m_of = {"none": lambda r: -1, "updown": lambda r: n - 1 - r, "given": lambda r: mate[r]}[mates]
    t = lambda a, dt: torch.as_tensor(a, dtype=dt).cuda()  # noqa: E731
    got = B.pair_reduce(n, t(ptr, torch.int64), t(np.append(pairs, 0), torch.int32),
                        t(np.concatenate([part, np.zeros((1, 12))]), torch.float32),
                        mate=t(mate, torch.int64) if mates == "given" else None, updown=mates == "updown").cpu().numpy()
    for r in range(n):
        want, size = np.zeros(6), np.zeros(6)
        for row, c in ((r, 0), (m_of(r), 6)):
            if row >= 0:
                v = part[pairs[ptr[row]:ptr[row + 1]], c:c + 6].astype(np.float64)
                want, size = want + v.sum(0), size + np.abs(v).sum(0)
        assert (np.abs(got[r] - want) <= 1e-13 * size).all(), r


@pytest.mark.parametrize("width,height,tile_w,mirror", [(8, 8, 0, 0), (65, 33, 16, 0), (131, 120, 0, 2), (128, 128, 16, 1),
                                                        (160, 160, 16, 3), (288, 288, 16, 3)])
def test_searched_against_sorted(width, height, tile_w, mirror):
    wl = W.config1()
    off_centre = 0 if mirror else 60  # a single tile at the centre sees nothing
    wl = dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, width=width, height=height, center_x=width / 2 - off_centre,
                                                          center_y=height / 2 - off_centre, tile_w=tile_w, mirror=mirror))
    eng = AG.PatternEngine(wl)
    a = wl.atoms
    atoms = eng.atoms(*(torch.as_tensor(v) for v in (a.x, a.y, a.z, a.B, a.occ)))
    F, F2 = B.structure_factors(eng.cell, atoms, eng.hkl)
    eng.plan.run(eng.hkl, F2)
    G = torch.as_tensor(np.random.default_rng(5).normal(size=(height, width)), dtype=torch.float32).cuda()
    model = eng.plan.model
    tx, ty = B.tile_grid(model.geom)
    n = int(eng.hkl.shape[0])
    print(f"{width}x{height}, {n} reflections, {tx * ty} tiles, {'searched' if n * tx * ty <= 1 << 25 else 'sorted'}", flush=True)
    out, glob, dF2 = B.pattern_backward(eng.plan, eng.hkl, F, G, atoms, deterministic=True)
    # the sorted route, step by step
    refl, cull = B.reflection_prep(model, eng.hkl, F2)
    nodes = B.node_table(model)
    pix, tile = B.pixel_map(model.geom)
    off, idx = B.cull(model.geom, tile, cull)
    part = torch.zeros((int(idx.numel()) + 1, 12), dtype=torch.float32, device="cuda")
    p = B._ptr
    B._check(B.lib().fdtbx_profile_adjoint_pairs(ctypes.byref(model), p(refl), p(nodes), p(pix), p(tile), p(off), p(idx), None, n,
                                                 int(idx.numel()), p(G), p(part), B._stream()))
    ptr, pairs = B.pair_transpose(n, idx)
    sums = B.pair_reduce(n, ptr, pairs, part, updown=bool(mirror & 2))
    want_f2, want_g = B.adjoint_finish(model, eng.hkl, refl, sums, F)
    scale = want_f2.abs().max().item()
    assert scale > 0
    assert (dF2 - want_f2).abs().max().item() <= 2.0 ** -23 * scale
    assert (glob - want_g).abs().max().item() <= 1e-9 * want_g.abs().max().item()
    again, glob2, dF22 = B.pattern_backward(eng.plan, eng.hkl, F, G, atoms, deterministic=True)
    assert torch.equal(dF2, dF22) and torch.equal(glob, glob2) and all(torch.equal(out[k], again[k]) for k in out)
