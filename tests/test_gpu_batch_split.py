"""The batched structure factors and their adjoint on both sides of the block counts at which
sixteen, four or one thread share a sum (64 and 256 blocks): batches of copies of two small
models, one with atoms and reflections that fill no block and one with more than a block of
each, must give every copy the values it has in a batch of the two alone, which run with sixteen.
Both sum in binary64, so the float32 values agree to a rounding (2^-22 of a group's largest)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_23245_amd.batch import BatchEngine  # noqa: E402


def run(n):
    wls = [W.small(51, n_atoms=23, width=16, height=16, n_nodes=4, d_min=6.0),
           W.small(52, n_atoms=270, width=16, height=16, n_nodes=4, d_min=2.2)]
    be = BatchEngine([wls[i % 2] for i in range(n)])
    be.forward()
    G = torch.ones_like(be.image)
    grads, glob = be.backward(G)
    torch.cuda.synchronize()
    print(f"{n} models: {int(be.refl_blocks.shape[0])} reflection blocks, {int(be.atom_blocks.shape[0])} atom blocks", flush=True)
    return be.F.clone(), {k: v.clone() for k, v in grads.items()}, glob.clone()


def close(a, b, what):
    assert b.abs().max() > 0, what
    assert (a - b).abs().max().item() <= 2.0 ** -22 * b.abs().max().item(), what


@pytest.mark.parametrize("n", [1, 3, 42, 44, 170, 172])
def test_copies_agree_with_the_pair(n):
    F0, g0, G0 = run(2)
    F, g, G = run(n)
    rest = {k: v.reshape(-1) for k, v in g.items()}
    pos = {k: 0 for k in g}
    at = 0
    one = F0.shape[0]
    first = run(1)[0].shape[0]  # reflections of the first model
    for i in range(n):
        lo, hi = (0, first) if i % 2 == 0 else (first, one)
        close(F[at:at + hi - lo], F0[lo:hi], f"F of copy {i}")
        at += hi - lo
        for k, v in rest.items():
            a, b = (0, 23) if i % 2 == 0 else (23, 293)
            close(v[pos[k]:pos[k] + b - a], g0[k].reshape(-1)[a:b], f"d{k} of copy {i}")
            pos[k] += b - a
        close(G[i], G0[i % 2], f"globals of copy {i}")
    assert at == F.shape[0]
