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


def batch_of(shapes, **kw):
    from paper_2608_23245_amd.batch import BatchEngine
    wls = [W.small(90 + i, width=w, height=h, center=(w / 2, h / 2), sigma_theta=0.05, gamma_theta=0.02, n_nodes=10, **kw)
           for i, (w, h) in enumerate(shapes)]
    return wls, BatchEngine(wls)


@pytest.mark.parametrize("unit", [1, 3, 64, 65, 100000])
def test_batch_units_match_whole_lists(unit):
    """The batched forward in units of one pair up to more than the longest list, lists of an odd
    number of tile rows and of none among them, against the launch with one wave per list: the
    same terms grouped otherwise (2e-6 of each model's largest value)."""
    _, eng = batch_of([(40, 37), (17, 9), (64, 64)])
    print(f"batch units of {unit}", flush=True)
    eng.forward()
    lens = np.zeros(int(eng.stack_items.shape[0]), dtype=np.int64)
    off, rp = eng.stack_off.cpu().numpy().reshape(-1, 3), eng.srowptr.cpu().numpy()
    for k, packed in enumerate(eng.stack_items.cpu().numpy()):
        m, s = int(packed >> 40), int(packed & ((1 << 40) - 1))
        lens[k] = rp[off[m, 1] + s + 1] - rp[off[m, 1] + s]
    n = -(-lens // unit)
    ptr = torch.as_tensor(np.concatenate([[0], np.cumsum(n)]), dtype=torch.int64).cuda()
    item = torch.as_tensor(np.repeat(np.arange(n.shape[0]), n), dtype=torch.int32).cuda()
    sums = torch.full((max(int(n.sum()), 1), 128), float("nan"), device="cuda")
    got, want = torch.full_like(eng.image, 7.0), torch.full_like(eng.image, 9.0)
    p = B._ptr
    tail = (p(eng.refl), p(eng.nodes), p(eng.pix), p(eng.tile), p(eng.stile), p(eng.srowptr), p(eng.sidx))
    head = (p(eng.entries), eng.n, p(eng.stack_off), p(eng.stack_items), int(eng.stack_items.shape[0]))
    B._check(B.lib().fdtbx_batch_profile_units(*head, p(ptr), p(item), int(n.sum()), unit, *tail, p(got), p(sums),
                                               B._stream()))
    B._check(B.lib().fdtbx_batch_profile_stacked(*head, *tail, p(want), p(eng.counter), B._stream()))
    for m in range(eng.n):
        s = slice(eng.pix_off[m], eng.pix_off[m + 1])
        assert (got[s] - want[s]).abs().max().item() <= 2e-6 * want[s].abs().max().item()
    assert B.lib().fdtbx_batch_profile_units(*head, p(ptr), p(item), int(n.sum()), 0, *tail, p(got), p(sums),
                                             B._stream()) == -1


@pytest.mark.parametrize("side", [88, 728])
def test_batch_adjoint_parts(side):
    """The batched adjoint with lists in 64 parts (121 tiles) and in 16 (8281 tiles) against the
    single-model launch: every pair's sums are the same, added in another order (the single
    launch's images are walked with wider node windows, which adds nothing but zeros)."""
    wls, eng = batch_of([(side, side)], d_min=4.0, distance=60.0 * side / 24)
    print(f"batch adjoint, {eng.items.shape[0]} items", flush=True)
    eng.forward()
    G = torch.as_tensor(np.random.default_rng(5).normal(size=side * side), dtype=torch.float32).cuda()
    eng.backward(G)
    model = eng.models[0]
    off = eng.rowptr
    want = B.profile_adjoint(model, eng.refl, eng.nodes, eng.pix, eng.tile, off, eng.idx, G.view(side, side))
    s = want.abs().amax(dim=0).clamp(min=1e-300)
    assert ((eng.sums - want).abs() / s).max().item() <= 1e-6


@pytest.mark.parametrize("lineshape", [0, 1, 2])
@pytest.mark.parametrize("n_nodes", [51, 52])
def test_split_and_unsplit_walk(lineshape, n_nodes):
    """The balanced launch on both sides of the node count from which its walk is split in two
    queues, against the per-tile launch (whose walk always is): the same terms, two queues' block
    sums against one's (2e-6 of the largest value)."""
    wl = W.small(95, width=33, height=26, sigma_theta=0.05, gamma_theta=0.02, n_nodes=n_nodes, lineshape=lineshape)
    model = B.make_model(wl)
    hkl = B.enumerate_hkl(model.cell, wl.quad.d_min, wl.quad.d_max)
    _, F2 = B.structure_factors(model.cell, atoms_to_device(wl.atoms), hkl, want_F=False)
    refl, cull = B.reflection_prep(model, hkl, F2)
    nodes = B.node_table(model)
    pix, tile = B.pixel_map(model.geom)
    off, idx = B.cull(model.geom, tile, cull)
    print(f"split walk, lineshape {lineshape}, {n_nodes} nodes: {idx.numel()} pairs", flush=True)
    img = B.profile_balanced(model, refl, nodes, pix, tile, off, idx)
    ref = B.profile(model, refl, nodes, pix, tile, off, idx)
    assert ref.max().item() > 0 and (img - ref).abs().max().item() <= 2e-6 * ref.max().item()
