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

from paper_2608_23245_amd.batch import BatchEngine  # noqa: E402


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
@pytest.mark.parametrize("stacked", [False])
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


@pytest.mark.parametrize("stacked", [False])
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
