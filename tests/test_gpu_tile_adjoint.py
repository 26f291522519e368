"""The backward pass of a 16-sequence tile (csrc/adj_mfma.hip, up to 48 states) against the
FP64 oracle, at the edges of its chunks and segments, of its partial of emission counts and of
its variants.

Tolerance.  A step of either recursion rounds at most 16 times (12 matrix products of 4 terms
in a row at 48 states, the emission product, the scale), each below 2^-24 of its value, and
no sequence has more than 100 steps before or after a count: 1.6e3 2^-24 = 1e-4 of each
sequence's counts, hence of their sums, which have no cancellation."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

TOL = 1e-4
EDGES = [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 15, 16, 17, 20, 24, 25, 26, 35, 36, 37, 49, 50, 63, 64, 65, 81, 99, 100]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    yield
    hmm.select_kernel(hmm.KERNEL_AUTO)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# One tile per CU (chunks of four steps at 16 states): small and large partials, the largest beside
# the ring of two steps, and sums in memory; then more tiles than CUs (chunks of two).
@pytest.mark.parametrize("N,M,S", [(1, 1, 90), (5, 6, 90), (16, 139, 90), (16, 140, 90), (16, 400, 90), (15, 800, 90),
                                   (16, 1200, 90), (16, 2300, 90), (9, 2400, 90), (17, 30, 90), (32, 150, 90),
                                   (31, 500, 90), (32, 1100, 90), (32, 1200, 90), (33, 20, 90), (48, 100, 90),
                                   (47, 690, 90), (48, 720, 90), (4, 9, 5000), (16, 60, 9000), (7, 30, 13000),
                                   (13, 6, 17000), (20, 40, 9000), (32, 50, 13000), (40, 30, 9000)])
def test_counts_of_tiles(N, M, S):
    print(f"[case] tile adjoint N={N} M={M} S={S}", flush=True)
    rng = np.random.default_rng([83, N, M, S])
    few = S < 1000
    lengths = np.array(EDGES + [int(x) for x in rng.integers(1, 101 if few else 9, size=S - len(EDGES))], np.int32)
    w = workloads.random_lengths_workload(rng, K=3, N=N, M=M, lengths=rng.permutation(lengths), all_pairs=False, conc=0.5)
    weight = rng.uniform(0.25, 1.75, size=S).astype(np.float32)
    if M > 4:
        for s in range(0, S, 2):  # many slots of a tile on one symbol
            w.symbols[w.offsets[s]:w.offsets[s] + w.lengths[s]] = 3
        w.B[0, :, 4] = 0.0        # impossible in model 0: such a sequence takes no part
        w.B[0] /= w.B[0].sum(axis=1, keepdims=True)
        w.symbols[w.symbols == 4] = 0
        dead = int(np.flatnonzero((w.owner == 0) & (w.lengths >= 5))[0])
        w.symbols[w.offsets[dead] + 2] = 4
    B = w.B.astype(np.float32)
    p = hmm.Problem(dev(w.pi), dev(w.A), dev(B), dev(w.symbols), dev(w.offsets), dev(w.lengths), dev(w.owner),
                    max_len=100, total_symbols=w.total_symbols)
    hmm.select_kernel(hmm.KERNEL_BATCHED)
    got = [x.cpu().numpy().astype(np.float64) for x in hmm.forward_backward_grad(p, dev(weight))[1]]
    ref = O.counts(w.pi, w.A, B, w.symbols, w.offsets, w.lengths, w.owner, weight)[1:]
    for name, g, r in zip(("pi", "A", "B"), got, ref):
        for k in range(3):
            assert np.linalg.norm(g[k] - r[k]) <= TOL * np.linalg.norm(r[k]), (name, k)
