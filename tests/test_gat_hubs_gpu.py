"""Attention over hubs, whose rows are folded from thousands of pieces: how far
the hub's own results are from 64 bits, per array (2-norm over 2-norm). A sum of
n rounded terms in k-term chains is about sqrt(k) 2^-25 of their magnitude off;
one chain over all pieces of a hub shows here, an elementwise bound scaled by
the sum of magnitudes does not."""
import numpy as np
import pytest
import torch

from tests.parity import to_dev
from tests.test_gat_fused_gpu import reference

pytestmark = pytest.mark.gpu


def rel(got, ref):
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("M", [3000, 150_000])  # hub edges: 47 and 2,344 pieces of 64 slots
@pytest.mark.parametrize("H,C", [(4, 4), (2, 32)])  # one and two groups of 64 columns in the gradient's fold
def test_gat_hub_error(M, H, C):
    import paper_1903_02428_amd as pyg
    N, S = 3000, 40 * 3000
    rng = np.random.default_rng(9100 + M + C)
    u = lambda n: rng.integers(0, N, n)
    a, b = N // 2, N // 3  # a: a hub of targets, b: a hub of sources
    ei = np.stack([np.concatenate([u(S), u(M), np.full(M, b)]), np.concatenate([u(S), np.full(M, a), u(M)])])
    # like-signed rows: the hub's sums do not cancel
    x = (rng.random((N, H * C)) + 0.5).astype(np.float32)
    g = (rng.random((N, H * C)) + 0.5).astype(np.float32)
    a_src, a_dst = (rng.standard_normal((N, H)).astype(np.float32) for _ in range(2))
    dev = [to_dev(t).requires_grad_(True) for t in (x, a_src, a_dst)]
    out = pyg.GATAttention.apply(*dev, pyg.Graph(to_dev(ei), N), 0.2)
    grads = torch.autograd.grad(out, dev, to_dev(g))
    torch.cuda.synchronize()
    ref = reference(x, a_src, a_dst, ei, g, 0.2)
    got = {n: t.detach().cpu().numpy() for n, t in zip(("out", "gx"), (out, grads[0]))}
    # chains of at most 16 slots, 16 pieces and a quarter of the pieces by 16
    # (37): 3e-7 is five times sqrt(40) 2^-25 / sqrt(12)
    assert rel(got["out"][a], ref["out"][0][a]) < 3e-7
    assert rel(got["gx"][b], ref["gx"][0][b]) < 3e-7


@pytest.mark.parametrize("H,C", [(8, 32), (2, 128)])  # 64 lanes a slot: one sub-group
def test_gat_long_row_error(H, C):
    # rows of about 800 slots that are reduced whole (chunks of 1,024): the
    # softmax's sum and the features' sums in chains of 8 and 25, where one chain
    # is 200 long: sqrt(200 / 33) or 2.5 times as far from 64 bits. The chains
    # give out 3.3e-7 and 1.7e-7.
    import paper_1903_02428_amd as pyg
    R, N = 96, 4000
    rng = np.random.default_rng(9200 + H)
    deg = rng.integers(780, 820, R)
    ei = np.stack([rng.integers(0, N, deg.sum()), np.repeat(np.arange(R), deg)])
    x, g = (rng.standard_normal((N, H * C)).astype(np.float32) for _ in range(2))
    a_src, a_dst = (rng.standard_normal((N, H)).astype(np.float32) for _ in range(2))
    dev = [to_dev(t).requires_grad_(True) for t in (x, a_src, a_dst)]
    graph = pyg.Graph(to_dev(ei), N)
    graph.csr.chunk = graph.csr_t.chunk = 1024
    out = pyg.GATAttention.apply(*dev, graph, 0.2)
    grads = torch.autograd.grad(out, dev, to_dev(g))
    torch.cuda.synchronize()
    ref = reference(x, a_src, a_dst, ei, g, 0.2)
    assert rel(out.detach().cpu().numpy()[:R], ref["out"][0][:R]) < 2.5e-7
    assert rel(grads[2].cpu().numpy()[:R], ref["gd"][0][:R]) < 8.5e-7
