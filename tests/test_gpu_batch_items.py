"""Batched launches over more items than one row of workgroups holds.  HIP refuses 2^32 threads
along one dimension and of more runs the excess alone, without an error: 2^22 items of sixteen
64-thread workgroups in the backward pass, 2^26 items of one in the forward's unit sums.  The items of a small batch are followed by copies of an item whose
list is empty until the count stands at that limit, one less or one more: the pass must be accepted
and give what the plain items give (an empty list adds nothing to a sum, and its pixels are zero)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd.batch import BatchEngine  # noqa: E402


def engine():
    """A model that is reached and one (the last, with empty lists) that is not."""
    be = BatchEngine([W.small(81), W.small(82, width=8, height=8, center=(-400.0, -400.0))], deterministic=True)
    assert be.list_len[0] > 0 and be.list_len[1] == 0
    return be


def with_copies(items, n):
    last = items[-1:]  # the shortest list
    return torch.cat([items, last.expand(n - items.shape[0])]).contiguous()


@pytest.mark.parametrize("n", [(1 << 22) - 1, 1 << 22, (1 << 22) + 1])
def test_backward(n):
    be = engine()
    be.forward()
    G = torch.as_tensor(np.random.default_rng(3).normal(size=be.image.numel()), dtype=torch.float32).cuda()
    be.items = with_copies(be.items, 8200)  # as many as are cut in sixteen
    want, want_g = be.backward(G)
    want, want_g = {k: v.clone() for k, v in want.items()}, want_g.clone()
    assert want_g.abs().max() > 0
    be.items = with_copies(be.items, n)
    print(f"{n} items", flush=True)
    for t in (*be.grads.values(), be.d_globals, be.partials):
        t.fill_(-1.0)
    got, got_g = be.backward(G)
    torch.cuda.synchronize()
    assert torch.equal(got_g, want_g) and all(torch.equal(got[k], want[k]) for k in want)


@pytest.mark.parametrize("n", [1 << 26, (1 << 26) + 1])
def test_forward_unit_sums(n):
    be = engine()
    want = be.forward().clone()
    assert want.abs().max() > 0
    be.stack_items = with_copies(be.stack_items, n)
    be.unit_ptr = with_copies(be.unit_ptr, n + 1)
    be.image.fill_(-1.0)
    print(f"{n} items", flush=True)
    got = be.forward()
    torch.cuda.synchronize()
    assert torch.equal(got, want)


def test_forward_units_beyond_one_launch():
    """2^26 units of empty lists, 1024 to each of 65536 items of a tile that nothing reaches, before the
    batch's own: those are then in the second of two launches (34 GB of unit sums)."""
    be = engine()
    want = be.forward().clone()
    empty = be.stack_items[-1:]
    assert be.unit_ptr[-1] == be.unit_ptr[-2] == be.n_units
    ahead = torch.arange(0, 1 << 26, 1024, device="cuda")
    be.stack_items = torch.cat([empty.expand(1 << 16), be.stack_items]).contiguous()
    be.unit_ptr = torch.cat([ahead, be.unit_ptr + (1 << 26)]).contiguous()
    be.unit_item = torch.cat([torch.arange(1 << 16, dtype=torch.int32, device="cuda").repeat_interleave(1024),
                              be.unit_item + (1 << 16)]).contiguous()
    be.n_units += 1 << 26
    be.unit_sums = torch.empty((be.n_units, 128), dtype=torch.float32, device="cuda")
    be.image.fill_(-1.0)
    print(f"{be.n_units} units", flush=True)
    got = be.forward()
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    be.unit_sums = None
    torch.cuda.empty_cache()
