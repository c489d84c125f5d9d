"""Batches with empty culling lists: a detector out of reach of every reflection is a valid
model.  Its image and all its gradients are exactly zero (sums over no pair), alone in a batch,
where no list holds a pair, and beside a model that is reached, whose image and gradients keep
the bits they have alone."""
import dataclasses

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd import binding as B  # noqa: E402
from paper_2608_23245_amd.batch import BatchEngine, GraphStep  # noqa: E402


def unreached(seed, **geom):
    """The beam 400 pixels outside the detector: every pixel beyond the resolution limit."""
    wl = W.small(seed, width=18, height=13, center=(-400.0, -400.0))
    return dataclasses.replace(wl, geom=dataclasses.replace(wl.geom, **geom))


def step(wls, **kw):
    be = BatchEngine(wls, **kw)
    be.image.fill_(-1.0)
    img = be.forward().clone()
    grads, glob = be.backward(torch.ones_like(img))
    torch.cuda.synchronize()
    return be, img, {k: v.clone() for k, v in grads.items()}, glob.clone()


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("stacked", [True, False])
@pytest.mark.parametrize("n", [1, 3])
def test_no_list_holds_a_pair(n, stacked, deterministic):
    be, img, grads, glob = step([unreached(70 + i, tile_w=(0, 16)[i % 2]) for i in range(n)], stacked=stacked,
                                deterministic=deterministic)
    print(f"{n} models, stacked {stacked}, fixed order {deterministic}: {be.list_len} pairs", flush=True)
    assert sum(be.list_len) == 0 and int(be.hkl.shape[0]) > 0
    assert img.shape == (n * 18 * 13,) and torch.count_nonzero(img).item() == 0
    assert torch.count_nonzero(glob).item() == 0
    for k, v in grads.items():
        assert torch.count_nonzero(v).item() == 0, k


@pytest.mark.parametrize("stacked", [True, False])
def test_beside_a_model_that_is_reached(stacked):
    full = W.small(75)
    _, img1, g1, glob1 = step([full], stacked=stacked, deterministic=True)
    be, img, g, glob = step([unreached(76), full, unreached(77)], stacked=stacked, deterministic=True)
    assert img1.abs().max() > 0 and be.list_len[0] == be.list_len[2] == 0
    at = 18 * 13
    assert torch.equal(img[at:at + img1.numel()], img1)
    assert torch.count_nonzero(img).item() == torch.count_nonzero(img1).item()
    assert torch.equal(glob[1], glob1[0]) and torch.count_nonzero(glob[[0, 2]]).item() == 0
    for k in g:
        assert torch.equal(g[k][be.atom_off[1]:be.atom_off[2]], g1[k]), k


def test_empty_batch_in_a_graph():
    be = BatchEngine([unreached(78)])
    gs = GraphStep(be, torch.full_like(be.image, 0.5))
    gs.capture()
    for _ in range(3):
        be.image.fill_(-1.0)
        be.d_globals.fill_(-1.0)
        gs.replay()
        torch.cuda.synchronize()
        assert torch.count_nonzero(be.image).item() == 0 and torch.count_nonzero(be.d_globals).item() == 0


def test_units_entry_without_units():
    """No unit: neither a unit table nor its sums nor a list are needed, and the items' pixels
    are written as zeros; with units their pointers are required."""
    be = BatchEngine([unreached(79)])
    be.image.fill_(-1.0)
    p = B._ptr

    def call(n_units):
        return B.lib().fdtbx_batch_profile_units(
            p(be.entries), be.n, p(be.stack_off), p(be.stack_items), int(be.stack_items.shape[0]), p(be.unit_ptr), None, n_units,
            be.unit_pairs, p(be.refl), p(be.nodes), p(be.pix), p(be.tile), p(be.stile), p(be.srowptr), None, p(be.image), None,
            B._stream())

    assert call(1) == -1  # FDTBX_ERR_INVALID_ARGUMENT, before any launch
    torch.cuda.synchronize()
    assert bool((be.image == -1.0).all())
    assert call(0) == 0
    torch.cuda.synchronize()
    assert torch.count_nonzero(be.image).item() == 0
