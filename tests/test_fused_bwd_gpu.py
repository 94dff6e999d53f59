"""The one-pass gradients (both gradients of a weighted or edge-feature
propagate over the reversed graph) against the separate kernels, bit for bit:
one lane to a whole wavefront per row, fewer lanes than slots in flight, rows
around a batch of 64 slots, long rows in pieces, empty rows, short rows on
sub-groups and long rows on whole wavefronts."""
import numpy as np
import pytest
import torch

import synth
from tests.parity import to_dev

pytestmark = pytest.mark.gpu

F32, BF16 = torch.float32, torch.bfloat16
# (N, E, F in 16-byte vectors, hub)
CASES = [(1, 1, 1, False), (50, 333, 1, False), (300, 9000, 2, True), (140, 140 * 139 // 2, 5, False), (4000, 30000, 16, True),
         (257, 6000, 25, False), (90, 5000, 64, True), (20000, 9000, 33, False)]


@pytest.fixture(scope="module")
def pyg():
    import paper_1903_02428_amd as m
    assert torch.cuda.is_available()
    m.library()
    return m


def build(pyg, case, dtype, seed, weighted):
    N, E, nv, hub = case
    rng = np.random.default_rng(seed)
    ei = synth.random_coo(rng, N, E)
    if hub:
        ei[1, : E // 2] = N // 2
        ei[0, E // 2:] = N // 3
    if N == 140:  # out-degrees 0 .. 139
        ei[0] = np.repeat(np.arange(N), np.arange(N))
    ei = to_dev(ei)
    F = nv * (4 if dtype == F32 else 8)
    w = to_dev(rng.standard_normal(E).astype(np.float32)) if weighted else None
    draw = lambda *s: to_dev(rng.standard_normal(s).astype(np.float32)).to(dtype)
    return (N, E, F, ei, w, pyg.coo_to_csr(ei, N, w), pyg.coo_to_csr(pyg.reverse_edges(ei), N, w), draw(N, F),
            draw(N, F), draw(E, F))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("aggr", ["sum", "mean"])
@pytest.mark.parametrize("case", CASES)
def test_weighted_one_pass_bits(pyg, case, aggr, dtype):
    N, E, F, ei, w, csr, csr_t, x, g, _ = build(pyg, case, dtype, 6000 + case[1], True)
    gx, gw = pyg.propagate_backward(g, x, ei, w, csr, csr_t, aggr, need_grad_w=True)
    px, pw = pyg.propagate_backward(g, x, ei, w, csr, csr_t, aggr, need_grad_w=True, w_order="csr")  # two passes
    assert torch.equal(gx, px) and torch.equal(gw[csr.perm], pw)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("aggr", ["sum", "mean"])
@pytest.mark.parametrize("msg", ["edge_add", "edge_relu", "edge_mul"])
@pytest.mark.parametrize("case", CASES)
def test_edge_one_pass_bits(pyg, case, msg, aggr, dtype):
    N, E, F, ei, _, csr, csr_t, x, g, ea = build(pyg, case, dtype, 6100 + case[1], False)
    a = (g, x, ea, csr, msg, aggr, "coo", csr_t)
    gx, ge = pyg.propagate_edge_backward(*a)
    px, _ = pyg.propagate_edge_backward(*a, need_grad_edge=False)
    _, pe = pyg.propagate_edge_backward(*a, need_grad_x=False)
    assert torch.equal(gx, px) and torch.equal(ge, pe)
