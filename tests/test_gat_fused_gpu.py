"""GPU parity of the one-pass attention kernels (pyg_gat_forward and
pyg_gat_backward through GATAttention) against the oracle's softmax, attention
sum and their gradients, where the kernels can go wrong: one slot, rows around
a batch of 64 and around a chunk, long rows folded from many pieces, short
rows on sub-groups, runs of empty rows, every split of lanes over heads,
several windows of heads, masked (-inf) and lowest logits."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import bf16_round, to_dev

pytestmark = pytest.mark.gpu

# (N, E, H, C, hub): lanes per head 1 .. 64 (fp32), one and several windows
CASES = [(1, 1, 1, 4, False), (9, 3, 2, 8, False), (300, 700, 8, 8, False), (64, 6000, 8, 16, False),
         (700, 20000, 4, 32, True), (5, 9000, 3, 8, True), (400, 5000, 1, 256, False), (257, 4000, 16, 32, True),
         (40, 5000, 2, 128, False), (90000, 70000, 4, 4, False)]


@pytest.fixture(scope="module")
def pyg():
    import paper_1903_02428_amd as m
    assert torch.cuda.is_available()
    m.library()
    return m


def reference(x, a_src, a_dst, ei, g, slope):
    """Forward and gradients in 64 bits by the oracle's separate steps, with
    the sums of magnitudes that scale the rounding of each result."""
    N, H = a_src.shape
    src, dst = ei
    C = x.shape[1] // H
    v = a_src[src].astype(np.float64) + a_dst[dst]
    e = np.where(v >= 0, v, slope * v)
    al = oracle.segment_softmax(e, ei, N)
    x64, g64 = x.astype(np.float64).reshape(N, H, C), g.astype(np.float64).reshape(N, H, C)

    def add(idx, val, n=N):
        o = np.zeros((n,) + val.shape[1:])
        np.add.at(o, idx, val)
        return o
    out = add(dst, al[..., None] * x64[src])
    s_out = add(dst, al[..., None] * np.abs(x64[src]))
    gx = add(src, al[..., None] * g64[dst])
    s_gx = add(src, al[..., None] * np.abs(g64[dst]))
    ga = (g64[dst] * x64[src]).sum(2)
    sa = (np.abs(g64[dst]) * np.abs(x64[src])).sum(2)
    t, st = add(dst, al * ga), add(dst, al * sa)
    d = np.where(v >= 0, 1.0, slope)
    dv, sv = al * (ga - t[dst]) * d, al * (sa + st[dst])
    return {"out": (out.reshape(N, -1), s_out.reshape(N, -1)), "gx": (gx.reshape(N, -1), s_gx.reshape(N, -1)),
            "gs": (add(src, dv), add(src, sv)), "gd": (add(dst, dv), add(dst, sv))}


def check(pyg, x, a_src, a_dst, ei, g, slope, dtype, msg):
    N = x.shape[0]
    dev = [to_dev(t) for t in (x, a_src, a_dst)]
    dev[0] = dev[0].to(dtype)
    for t in dev:
        t.requires_grad_(True)
    graph = pyg.Graph(to_dev(ei), N)
    out = pyg.GATAttention.apply(*dev, graph, slope)
    assert graph._map_t is None  # the one-pass kernels ran: no transpose map was needed
    grads = torch.autograd.grad(out, dev, to_dev(g).to(dtype))
    assert graph._map_t is None
    torch.cuda.synchronize()
    ref = reference(x, a_src, a_dst, ei, g, slope)
    # exp(s - m) by the hardware exp2 and rounded scores: 2^-24 of the largest
    # |score| per factor, beside the 1e-5 of every fp32 sum
    fin = np.concatenate([a[np.abs(a) < 1e30] for a in (a_src, a_dst)])
    rel = 2e-5 + 8 * 2.0 ** -24 * (1 + 2 * max(1.0, abs(slope)) * np.abs(fin).max())
    for name, got in zip(("out", "gx", "gs", "gd"), (out, *grads)):
        val, mag = ref[name]
        tol = rel * mag + 1e-6
        if got.dtype == torch.bfloat16:
            tol = tol + 2.0 ** -8 * np.abs(val)  # one rounding to bf16
        err = np.abs(got.detach().float().cpu().numpy() - val)
        assert (err <= tol).all(), (msg, name, float((err - tol).max()))
    return out, grads


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("case", CASES)
def test_gat_fused_parity(pyg, case, dtype):
    N, E, H, C, hub = case
    if dtype == torch.bfloat16 and C % 8:
        C *= 2
    rng = np.random.default_rng(5000 + N + E)
    ei = synth.random_coo(rng, N, E)
    if hub:
        ei[1, : E // 2] = N // 2
        ei[0, E // 2:] = N // 3
    x, g = (rng.standard_normal((N, H * C)).astype(np.float32) for _ in range(2))
    if dtype == torch.bfloat16:
        x, g = bf16_round(x), bf16_round(g)
    a_src, a_dst = (rng.standard_normal((N, H)).astype(np.float32) for _ in range(2))
    check(pyg, x, a_src, a_dst, ei, g, 0.2, dtype, (N, E, H, C))


def test_gat_fused_rows_around_batches_and_chunks(pyg):
    # in- and out-degrees 1 .. 130 (batches of 64) and around the 64-slot
    # chunks of a graph of this size, heavy rows (mean above 16)
    rng = np.random.default_rng(5100)
    deg = np.concatenate([np.arange(131), [63, 64, 65, 127, 128, 129, 1000]])
    ei = synth.graded_in_degree(rng, 140, deg)
    ei = np.concatenate([ei, ei[::-1]], axis=1)
    N, H, C = 140, 4, 8
    x, g = (rng.standard_normal((N, H * C)).astype(np.float32) for _ in range(2))
    a_src, a_dst = (rng.standard_normal((N, H)).astype(np.float32) for _ in range(2))
    for slope in (0.2, 1.0, 0.0, -0.5):
        first = check(pyg, x, a_src, a_dst, ei, g, slope, torch.float32, slope)
        again = check(pyg, x, a_src, a_dst, ei, g, slope, torch.float32, slope)
        for p, q in zip((first[0], *first[1]), (again[0], *again[1])):
            assert torch.equal(p, q)  # fixed orders


def test_gat_fused_masked_and_lowest_logits(pyg):
    # -inf masks a source; the type's lowest value masks it unless every
    # source of a target has it
    rng = np.random.default_rng(5200)
    N, H, C = 200, 2, 8
    ei = synth.random_coo(rng, N, 4000)
    ei[0, ::5] = 0  # every row may meet the masked nodes
    ei = np.concatenate([ei, np.stack([np.full(N, N - 1), np.arange(N)])], axis=1)  # and one that is not
    x, g = (rng.standard_normal((N, H * C)).astype(np.float32) for _ in range(2))
    a_src, a_dst = (rng.standard_normal((N, H)).astype(np.float32) for _ in range(2))
    low = a_src.copy()
    low[: N // 2] = np.finfo(np.float32).min / 8
    ref = None
    for fill in (np.finfo(np.float32).min / 8, -np.inf):
        a = a_src.copy()
        a[: N // 2] = fill
        dev = [to_dev(t).requires_grad_(True) for t in (x, a, a_dst)]
        out = pyg.GATAttention.apply(*dev, pyg.Graph(to_dev(ei), N), 0.2)
        grads = torch.autograd.grad(out, dev, to_dev(g))
        got = [t.detach().cpu().numpy() for t in (out, *grads)]
        assert all(np.isfinite(t).all() for t in got)
        assert (got[1][: N // 2] == 0).all() and (got[2][: N // 2] == 0).all()
        ref = ref or got
        assert all(np.array_equal(p, q) for p, q in zip(ref, got))
    # a target whose sources all have the lowest value: uniform coefficients
    one = np.stack([np.arange(5), np.full(5, 5)])
    a = np.full((6, 1), np.finfo(np.float32).min / 8, np.float32)
    xs = rng.standard_normal((6, 4)).astype(np.float32)
    out = pyg.GATAttention.apply(to_dev(xs), to_dev(a), to_dev(np.zeros((6, 1), np.float32)),
                                 pyg.Graph(to_dev(one.astype(np.int64)), 6), 0.2)
    assert np.allclose(out.cpu().numpy()[5], xs[:5].mean(0), rtol=1e-5, atol=1e-6)


def test_gat_fused_takes_what_the_separate_kernels_took(pyg):
    # unaligned rows and head widths that are no vectors take the separate
    # kernels; an output changed in place keeps its gradient
    rng = np.random.default_rng(5300)
    N, H, C = 50, 2, 8
    ei = to_dev(synth.random_coo(rng, N, 400))
    graph = pyg.Graph(ei, N)
    buf = to_dev(rng.standard_normal(N * H * C + 1).astype(np.float32))
    xs = [buf[1:].view(N, H * C), buf[1:].view(N, H * C).clone()]
    logits = [to_dev(rng.standard_normal((N, H)).astype(np.float32)) for _ in range(2)]
    res = []
    for x in xs:
        x = x.detach().requires_grad_(True)
        out = pyg.GATAttention.apply(x, *logits, graph, 0.2)
        out.mul_(2.0)
        (gx,) = torch.autograd.grad(out.sum(), [x])
        res.append((out.detach(), gx))
    for p, q in zip(*res):
        assert torch.allclose(p, q, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_gat_fused_upstream_of_isolated_nodes(pyg, bad):
    # a node without incoming edges passes nothing back, whatever its upstream
    # gradient holds: an empty sum, as by the separate kernels
    rng = np.random.default_rng(5500)
    N, H, C = 60, 2, 8
    ei = synth.random_coo(rng, N, 500)
    ei[1] %= N // 2  # targets below N / 2
    x, g = (rng.standard_normal((N, H * C)).astype(np.float32) for _ in range(2))
    a_src, a_dst = (rng.standard_normal((N, H)).astype(np.float32) for _ in range(2))
    ref = None
    for fill in (0.0, bad):
        g[N // 2:] = fill
        dev = [to_dev(t).requires_grad_(True) for t in (x, a_src, a_dst)]
        out = pyg.GATAttention.apply(*dev, pyg.Graph(to_dev(ei), N), 0.2)
        got = torch.autograd.grad(out, dev, to_dev(g))
        assert (got[2][N // 2:] == 0).all()
        ref = ref or got
        assert all(torch.equal(p, q) for p, q in zip(ref, got))


def test_gat_fused_saved_tensor_hooks(pyg):
    # what hooks hand back to the gradient: host copies brought back, unaligned
    # and transposed copies (the same bits), and tensors that no kernel may read
    rng = np.random.default_rng(5400)
    N, H, C = 50, 2, 8
    graph = pyg.Graph(to_dev(synth.random_coo(rng, N, 400)), N)
    x, g = (to_dev(rng.standard_normal((N, H * C)).astype(np.float32)) for _ in range(2))
    logits = [to_dev(rng.standard_normal((N, H)).astype(np.float32)) for _ in range(2)]

    def grads(hooks):
        dev = [t.detach().clone().requires_grad_(True) for t in (x, *logits)]
        with hooks:
            out = pyg.GATAttention.apply(*dev, graph, 0.2)
        return torch.autograd.grad(out, dev, g)

    def unaligned(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        return buf[1:].view(t.shape).copy_(t)

    def strided(t):
        return t.transpose(0, 1).contiguous().transpose(0, 1)

    hook = torch.autograd.graph.saved_tensors_hooks
    ref = grads(hook(lambda t: t, lambda t: t))
    for h in (torch.autograd.graph.save_on_cpu(), hook(lambda t: t, unaligned), hook(lambda t: t, strided)):
        for p, q in zip(ref, grads(h)):
            assert torch.equal(p, q)
    # refused on the host, before any launch: another device, another type
    for bad in (lambda t: t.cpu(), lambda t: t.double()):
        with pytest.raises((ValueError, RuntimeError)):
            grads(hook(lambda t: t, lambda t, bad=bad: bad(t) if t.dim() == 3 else t))
