"""Segments of one to four steps in the backward pass of a 16-sequence tile (csrc/adj_mfma.hip):
each half of the segment buffer is written again as soon as its rows have been taken, every few
steps, and the counts must be those of the FP64 oracle and the same bits on every call.

Tolerance.  A step of either recursion rounds at most 16 times, each below 2^-24 of its value, and
no sequence has more than 16 steps before or after a count: 256 2^-24 = 1.6e-5 of each sequence's
counts, hence of their sums, which have no cancellation."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

TOL = 1.6e-5


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# one tile per CU and several, with the partial in LDS and with sums in memory
@pytest.mark.parametrize("N,M,S", [(5, 6, 200), (16, 40, 9000), (16, 2600, 200), (32, 30, 200), (31, 50, 9000),
                                   (32, 1300, 200), (48, 30, 200), (33, 20, 9000), (48, 900, 200)])
def test_short_segments(N, M, S):
    print(f"[case] short segments N={N} M={M} S={S}", flush=True)
    rng = np.random.default_rng([101, N, M, S])
    w = workloads.random_lengths_workload(rng, K=2, N=N, M=M, lengths=rng.integers(1, 17, size=S).astype(np.int32),
                                          all_pairs=False, conc=0.5)
    p = hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets), dev(w.lengths), dev(w.owner),
                    max_len=16, total_symbols=w.total_symbols)
    ws = p.workspace(hmm.OP_GRAD)
    ref = O.counts(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, w.owner)[1:]
    first = None
    for _ in range(8):
        got = [x.clone() for x in hmm.forward_backward_grad(p, ws=ws)[1]]
        if first is None:
            first = got
            for name, x, r in zip(("pi", "A", "B"), got, ref):
                x = x.cpu().numpy().astype(np.float64)
                for k in range(2):
                    assert np.linalg.norm(x[k] - r[k]) <= TOL * np.linalg.norm(r[k]), (name, k)
        for name, x, y in zip(("pi", "A", "B"), got, first):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), name
