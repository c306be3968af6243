"""The sums of the contractions over all modes but one (the numerators of a factor) run as chains of a
64th of their products and trees of those.  Shown by one large product among ones: what is added to the
chain or to a tree's node that holds it is lost in rounding.

With a zero first factor and identities as the others, the gradient of the first factor is minus the
contraction of X with the core; a rank above 32 in another mode takes the general path."""
import numpy as np
import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r0,r1,r2,n0", [(4, 33, 20, 64), (20, 34, 9, 97), (32, 40, 25, 64), (3, 33, 2, 64)])
def test_a_large_product_loses_few_of_the_others(r0, r1, r2, n0):
    nnc = need_gpu()
    total = r1 * r2
    per = -(-(-(-total // 4)) // 8)  # steps of four products a wave
    chain = 4 * -(-per // 8)
    big = 2.0 ** 24  # every addition to it rounds to even integers: off by 1 at most
    dev = "cuda"
    X = torch.ones(n0, r1, r2, device=dev)
    at = np.linspace(0, total - 1, n0).astype(int)
    X.view(n0, total)[torch.arange(n0), torch.from_numpy(at)] = big
    G = torch.ones(r0, r1, r2, device=dev)
    A = [torch.zeros(n0, r0, device=dev), torch.eye(r1, device=dev), torch.eye(r2, device=dev)]
    print("case", r0, r1, r2, n0, flush=True)
    _, _, g = nnc.nntucker_grad(X, G, A)
    off = (-g[0].double() - (big + total - 1)).abs()
    # the chain, a tree of eight of them and a tree of the eight waves' sums
    assert off.max().item() <= chain + 6, (off.max().item(), chain)


@pytest.mark.parametrize("r0", [2, 17])
def test_sums_of_more_than_two_to_the_22_products(r0):
    """The same over 33 x 50 x 50 x 52 products, past the indices that a float division splits."""
    nnc = need_gpu()
    n0, rest = 65, (33, 50, 50, 52)
    total = int(np.prod(rest))
    chain = 4 * -(-(-(-(-(-total // 4)) // 8)) // 8)
    X = torch.ones(n0, *rest, device="cuda")
    at = np.linspace(0, total - 1, n0).astype(int)
    X.view(n0, total)[torch.arange(n0), torch.from_numpy(at)] = 2.0 ** 24
    G = torch.ones(r0, *rest, device="cuda")
    print("case", r0, flush=True)
    _, _, g = nnc.nntucker_grad(X, G, [torch.zeros(n0, r0, device="cuda")] + [torch.eye(n, device="cuda") for n in rest])
    off = (-g[0].double() - (2.0 ** 24 + total - 1)).abs()
    assert off.max().item() <= chain + 6, (off.max().item(), chain)
