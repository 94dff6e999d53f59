"""Light rows that are left to the whole wavefront: rows just below, at and
above the sub-group limit (twice the mean, 16 to 32 slots), the chunk (64) and
its multiples, among short and empty rows, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import check_sum, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [300, 900, 3000])  # means that put the limit at 32, between and at 16
@pytest.mark.parametrize("F", [4, 32, 64, 128])  # 64 to 2 rows side by side
def test_mixed_light_rows(N, F):
    import paper_1903_02428_amd as pyg
    rng = np.random.default_rng(7400 + N + F)
    deg = np.concatenate([[15, 16, 17, 18, 31, 32, 33, 63, 64, 65, 127, 128, 129, 500], rng.integers(0, 8, 200)])
    ei = synth.graded_in_degree(rng, N, rng.permutation(deg))
    E = ei.shape[1]
    assert E <= 16 * N
    x = rng.standard_normal((N, F)).astype(np.float32)
    w = rng.standard_normal(E).astype(np.float32)
    csr = pyg.coo_to_csr(to_dev(ei), N, to_dev(w), chunk=64)
    plain = pyg.CSR(csr.rowptr, csr.col, csr.perm, None, N, E, 64)
    out, _ = pyg.propagate(to_dev(x), csr=csr, aggr="sum")
    mx, arg = pyg.propagate(to_dev(x), csr=plain, aggr="max")
    torch.cuda.synchronize()
    ref, _, s = oracle.propagate(x, ei, w, aggr="sum")
    check_sum(out, ref, s, False, f"light sum N={N} F={F}")
    rmx, rarg, _ = oracle.propagate(x, ei, aggr="max")
    assert np.array_equal(mx.cpu().numpy(), rmx.astype(np.float32)) and np.array_equal(arg.cpu().numpy(), rarg)
