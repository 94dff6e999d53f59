"""Folds of long rows from their pieces: rows of one piece more and less than
one wavefront folds (16) and than a batch in flight (8), hundreds of pieces,
feature counts around the 64 of a wavefront, one and several chunks per
wavefront, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests.parity import check_max, check_sum, to_dev

pytestmark = pytest.mark.gpu

CHUNK = 16
PIECES = [1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 18, 33, 63, 64, 65, 66, 300]


@pytest.mark.parametrize("N", [700, 60000])  # 750 chunks, 11,000 (several per wavefront from 64 features on)
@pytest.mark.parametrize("F", [1, 63, 64, 65, 128, 130, 260])
def test_fold_of_pieces(N, F):
    import paper_1903_02428_amd as pyg
    rng = np.random.default_rng(8100 + N + F)
    # a row of k pieces at any offset in its first chunk has 16 (k - 1) + 1 to 16 k slots
    deg = np.concatenate([[CHUNK * k - rng.integers(0, 8), CHUNK * k + 1] for k in PIECES])
    rest = rng.integers(0, 5, N - deg.size) if N > 1000 else np.zeros(N - deg.size, int)
    ei = synth.graded_in_degree(rng, N, rng.permutation(np.concatenate([deg, rest])))
    E = ei.shape[1]
    x = rng.standard_normal((N, F)).astype(np.float32)
    csr = pyg.coo_to_csr(to_dev(ei), N, chunk=CHUNK)
    got = {a: pyg.propagate(to_dev(x), csr=csr, aggr=a) for a in ("sum", "mean", "max")}
    torch.cuda.synchronize()
    for a, (out, arg) in got.items():
        ref, rarg, s = oracle.propagate(x, ei, aggr=a)
        if a == "max":
            check_max(out, arg, ref, rarg, False, f"N={N} F={F} E={E}")
        else:
            check_sum(out, ref, s, False, f"{a} N={N} F={F} E={E}")
